"""What a solve leaves behind when it returns: nothing in its stream."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2207_08716_amd import inputs, schedules

pytestmark = pytest.mark.gpu

STATE = ("vx", "vy", "vz", "pt", "pf", "rx", "ry", "rz")


def _grid(shape):
    nx, ny, nz = shape
    cfg = dataclasses.replace(inputs.config_mixed(nx), nx=nx, ny=ny, nz=nz)
    cfg.phys = cfg.phys.replace(nup=15)
    g = schedules.make_grid(cfg, inputs.initial_fields(cfg))
    g.begin_step(False)
    g.refresh(1.0, 1.0)
    return g


@pytest.mark.parametrize("static", [False, True])
def test_a_solve_at_its_limit_has_left_its_stream(static):
    # the first handle stops 3 sweeps past a check; those read the gate, which
    # in the static scratch lies under the second handle's partial maxima
    def solve(g, *args):
        return (g.solve_linear_static if static else g.solve_linear)(*args)

    alone = _grid((127, 127, 127))
    solve(alone, 1e-300, 18)
    with torch.cuda.stream(torch.cuda.Stream()):
        a = _grid((127, 127, 127))
    with torch.cuda.stream(torch.cuda.Stream()):
        b = _grid((150, 150, 150))
    torch.cuda.synchronize()
    assert solve(a, 1e-300, 18)[0] == 18
    assert solve(b, 1e-300, 30)[0] == 30
    torch.cuda.synchronize()
    for n in STATE:
        assert np.array_equal(a.get(n), alone.get(n)), n


def test_a_mixed_solve_that_diverges_has_left_its_stream():
    # the FP64 residual is finite; an FP32 coefficient that overflows makes
    # the first correction's norms non-finite
    g = _grid((127, 127, 127))
    kc = g.get("kc")
    kc[60, 61, 62] = 1e300
    g.set("kc", kc)
    with pytest.raises(Exception, match="non-finite"):
        g.solve_mixed(1e-8, 1e-2, 1000, 5)
    assert g.stream.query()


def test_destroying_a_handle_does_not_wait_for_another_stream():
    with torch.cuda.stream(torch.cuda.Stream()):
        a = _grid((21, 18, 15))
    with torch.cuda.stream(torch.cuda.Stream()):
        b = _grid((255, 255, 255))
    a.solve_linear(1e-300, 40)
    b.iterate(15)
    torch.cuda.synchronize()
    b.iterate(300)          # 0.2 s
    a.close()
    assert not b.stream.query()
    torch.cuda.synchronize()
