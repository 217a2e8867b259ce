"""Where a solve stops: the sweeps launched past the check that ended it leave
no trace, and the iteration counts are those at which the rule first holds."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08716_amd import inputs, schedules

pytestmark = pytest.mark.gpu

STATE = ("vx", "vy", "vz", "pt", "pf", "rx", "ry", "rz")


def _grid(nup, shape=(21, 18, 15)):
    nx, ny, nz = shape
    cfg = dataclasses.replace(inputs.config_mixed(nx), nx=nx, ny=ny, nz=nz)
    cfg.phys = cfg.phys.replace(nup=nup)
    g = schedules.make_grid(cfg, inputs.initial_fields(cfg))
    g.begin_step(False)
    g.refresh(1.0, 1.0)
    return g


def _same(a, b, names=STATE):
    for n in names:
        assert np.array_equal(a.get(n), b.get(n)), n


@pytest.mark.parametrize("nup", [1, 2, 15, 64])
@pytest.mark.parametrize("static", [False, True])
def test_linear_solve_stops_at_its_check(nup, static):
    a, b = _grid(nup), _grid(nup)
    solve = a.solve_linear_static if static else a.solve_linear
    it, rho, ok = solve(1e-3)
    assert ok and it % nup == 0 and it > 1
    n = a.counters().iter
    # the same sweeps with no check able to end them, the last one a check
    it_b, rho_b, ok_b = b.solve_linear(1e-300, it)
    assert it_b == it and rho_b == rho and not ok_b and b.counters().iter == n
    _same(a, b)
    if it > nup:
        # one check earlier the rule did not hold
        c = _grid(nup)
        assert c.solve_linear(1e-300, it - nup)[1] > 1e-3
    # and both go on alike
    for g in (a, b):
        g.set_residual_reference(None)
    assert a.solve_linear(1e-4, 7 * nup + 3)[:2] == b.solve_linear(1e-4, 7 * nup + 3)[:2]
    _same(a, b)


@pytest.mark.parametrize("eta_in", [1e-2, 1e-9])
def test_mixed_solve_stops_at_its_check(eta_in):
    # 1e-9 is below what an FP32 correction reaches: the stall rule ends it
    a, b = _grid(5), _grid(5)
    it, _, _ = a.solve_mixed(1e-300, eta_in, 100000, 1)[:3]
    it = int(it)
    assert it % 5 == 0 and 5 < it < 100000
    b.solve_mixed(1e-300, 1e-300, it, 1)
    _same(a, b, ("vx", "vy", "vz", "pt", "pf"))


def test_a_solve_that_diverges_reports_its_check():
    g = _grid(15)
    g.solve_linear(1e-300, 20)
    pt = g.get("pt")
    pt[3, 4, 5] = np.nan
    g.set("pt", pt)
    with pytest.raises(Exception, match="non-finite"):
        g.solve_linear(1e-300, 1000)
    # the solve's first check, not a later one
    assert g.counters().iter == 20 + 15
