"""Every tile of the sweeps (thesis, linear, FP32 correction, residual, with
and without norms) on grids whose size makes the launch rule choose it, with
ragged last tiles and chunks, against the FP64 oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2207_08716_amd import inputs, schedules

from test_gpu_parity import STATE, _compare, _pair

pytestmark = pytest.mark.gpu

# by the plain FP64 sweeps' tile: 34 x 4 (one plane per block, and two), 34 x 6
# (one plane, several), 34 x 14, 66 x 6, 66 x 10 (one chunk per block, several)
GRIDS = [(7, 9, 8), (16, 15, 13), (31, 27, 30), (33, 30, 21), (75, 61, 40), (47, 45, 49), (90, 60, 62), (40, 33, 50),
         (64, 57, 61), (110, 50, 75)]


def _cfg(shape, **phys):
    cfg = inputs.config_fp64_picard(8)
    nx, ny, nz = shape
    cfg = dataclasses.replace(cfg, nx=nx, ny=ny, nz=nz, name="tilings")
    cfg.phys = cfg.phys.replace(lx=nx / 40, ly=ny / 40, lz=nz / 40, **phys)
    return cfg


@pytest.mark.parametrize("shape", GRIDS)
def test_sweeps_match_the_oracle_on_every_tile(shape):
    g, o = _pair(_cfg(shape))
    g.begin_step(False)
    o.begin_step()
    g.refresh()
    o.refresh()
    for update, norms in ((True, False), (True, True), (True, False), (False, False), (False, True), (False, False)):
        g.iteration(update, norms)
        last = o.iteration(update, norms)
        if norms:
            # max norms of residuals and changes: differences of fields, each
            # within 1e-12 of its scale, over cells of size h
            got = g.last_norms()
            for k, v in zip(("f", "rpt", "rpf", "dl", "dpt", "dpf", "dvz", "dv"), last.values()):
                assert abs(got[k] - v) <= 1e-10 * max(abs(v), 1e-3), (k, got[k], v)
    _compare(g, o, STATE)


@pytest.mark.parametrize("shape", [(33, 30, 21), (47, 45, 49), (40, 33, 50)])
def test_background_shear_on_small_tiles(shape):
    nx, ny, nz = shape
    cfg = inputs.config_production(nx, ny, nz)
    g, o = _pair(cfg)
    g.begin_step(False)
    o.begin_step()
    g.iterate(32)
    o.iterate(32)
    _compare(g, o, STATE)


@pytest.mark.parametrize("shape", [(7, 9, 8), (33, 30, 21), (47, 45, 49), (64, 57, 61), (90, 60, 62)])
def test_residual_and_correction_on_small_tiles(shape):
    # the FP64 residual, and the mixed solve's FP32 sweeps on it: 45 sweeps of
    # a correction equal 45 linear FP64 sweeps to FP32 accuracy (rounding of
    # 6e-8 per sweep and value, a few per sweep, on the state's scale)
    g, o = _pair(_cfg(shape))
    g.begin_step(False)
    o.begin_step()
    g.refresh(1.0, 1.0)
    o.refresh(1.0, 1.0)
    g.residual()
    for got, ref in zip(g.residual_fields(), o.residual()):
        assert np.abs(got - ref).max() <= 1e-6 * max(np.abs(ref).max(), 1e-30)
    g.solve_mixed(1e-300, 1e-30, 45, 1)
    for _ in range(45):
        o.iteration(False)
    for n in ("vx", "vy", "vz", "pt", "pf"):
        ref = o.f[n]
        assert np.abs(g.get(n) - ref).max() <= 45 * 4 * 6e-8 * np.abs(ref).max(), n
