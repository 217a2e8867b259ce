"""Mechanics off (PT_F_MECHOFF): V, R and Pt keep their values bit for bit,
whatever the forces on them, and the rest of the step does not notice."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08716_amd import inputs, schedules

from test_gpu_parity import STATE, _compare, _pair

pytestmark = pytest.mark.gpu

FROZEN = ("vx", "vy", "vz", "rx", "ry", "rz", "pt")


def _grid(shape=(37, 21, 18)):
    nx, ny, nz = shape
    cfg = dataclasses.replace(inputs.config_mixed(nx), nx=nx, ny=ny, nz=nz)
    cfg.phys = cfg.phys.replace(mech_off=True, nup=3)
    g = schedules.make_grid(cfg, inputs.initial_fields(cfg))
    g.begin_step(False)
    g.refresh(1.0, 1.0)
    rng = np.random.default_rng(5)
    for n in FROZEN:
        v = g.get(n)
        ax = {"x": 2, "y": 1, "z": 0}.get(n[1] if n != "pt" else "")
        v[...] = 1e-3 * rng.standard_normal(v.shape)
        if ax is not None:   # walls hold zero
            v[(slice(None),) * ax + (0,)] = 0.0
            v[(slice(None),) * ax + (-1,)] = 0.0
        g.set(n, v)
    return g


def _spoil(g, what):
    if what == "force":
        for n in ("fox", "foy", "foz"):
            f = g.get(n)
            f[7, 8, 9], f[7, 8, 11] = np.inf, np.nan
            g.set(n, f)
    else:                       # a divergence that overflows
        v = g.get("vx")
        v[7, 8, 9], v[7, 8, 10] = -1.5e308, 1.5e308
        g.set("vx", v)


@pytest.mark.parametrize("what,update_lp", [("force", True), ("force", False), ("velocity", False)])
def test_frozen_fields_stay(what, update_lp):
    a, b = _grid(), _grid()
    _spoil(a, what)
    before = {n: a.get(n) for n in FROZEN}
    for it in range(4):
        for g in (a, b):
            g.iteration(update_lp, norms=it == 2)
    for n in FROZEN:
        assert np.array_equal(a.get(n), before[n]), n
    for n in ("pf", "lp"):
        assert np.array_equal(a.get(n), b.get(n)) and np.isfinite(a.get(n)).all(), n
    assert not np.array_equal(b.get("pf"), _grid().get("pf"))


def test_frozen_multigrid_cycles_stay_finite():
    # V, R and Pt of every grid of the hierarchy are frozen too, the coarsest's
    # own kernel included: infinite forces reach neither Pf nor V
    a, b = _grid((32, 32, 32)), _grid((32, 32, 32))
    for n in ("fox", "foy", "foz"):
        f = a.get(n)
        f[7, 8, 9] = 1e300      # finite in FP64, infinite in the FP32 residual
        a.set(n, f)
    before = {n: a.get(n) for n in FROZEN}
    for g in (a, b):
        g.set_residual_reference((1.0, 1.0))
        g.solve_mg(1e-300, 2)
    for n in ("vx", "vy", "vz", "pt"):
        assert np.array_equal(a.get(n), before[n]), n
    assert np.array_equal(a.get("pf"), b.get("pf")) and np.isfinite(a.get("pf")).all()


@pytest.mark.parametrize("shape", [(7, 9, 8), (33, 30, 21), (75, 61, 40), (47, 45, 49), (64, 57, 61), (110, 50, 75),
                                   (108, 34, 364), (48, 123, 227)])
@pytest.mark.parametrize("shear", [0.0, 0.7])
def test_frozen_sweeps_match_the_oracle_on_every_tile(shape, shear):
    nx, ny, nz = shape
    cfg = dataclasses.replace(inputs.config_fp64_picard(8), nx=nx, ny=ny, nz=nz, name="frozen")
    cfg.phys = cfg.phys.replace(lx=nx / 40, ly=ny / 40, lz=nz / 40, mech_off=True, shear_bg=shear)
    g, o = _pair(cfg)
    for x in (g, o):
        x.begin_step(*([False] if x is g else []))
        x.refresh()
    for update, norms in ((True, False), (True, True), (True, False), (False, False), (False, True), (False, False)):
        g.iteration(update, norms)
        o.iteration(update, norms)
    _compare(g, o, STATE)
