"""The sweeps of grids whose fields outgrow the last-level cache, on each tile
that the rule sends such grids to, ragged, with chunks of an even and an odd
number of planes."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from test_gpu_parity import STATE, _compare, _pair
from test_gpu_tilings import _cfg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# grid: tile width, height, planes per chunk (of the plain FP64 sweeps)
FP64 = {(108, 34, 364): (34, 14, 18), (70, 95, 202): (34, 14, 21), (125, 44, 244): (66, 10, 12), (48, 123, 227): (66, 10, 15)}
# (of the FP32 correction sweeps)
FP32 = {(92, 135, 249): (34, 14, 36), (71, 112, 386): (34, 14, 23), (111, 145, 205): (66, 10, 16), (123, 74, 343): (66, 10, 29),
        (97, 81, 392): (66, 14, 22), (127, 184, 131): (66, 14, 17)}
CACHED64, CACHED32 = 256e6 / 192, 256e6 / 84      # cells


def test_the_grids_reach_every_tile(tmp_path):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "probe")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2207_08716_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tiling_probe.hip"), "-o", exe], check=True, capture_output=True)

    def tiles(shapes, kind):
        out = subprocess.run([exe, *[str(v) for s in shapes for v in s]], check=True, capture_output=True, text=True).stdout
        rows = [tuple(map(int, line.split())) for line in out.splitlines()]
        return {r[:3]: r[4:7] for r in rows if r[3] == kind}

    assert tiles(FP64, 0) == FP64 and all(np.prod(s) > CACHED64 for s in FP64)
    assert tiles(FP32, 1) == FP32 and all(np.prod(s) > CACHED32 for s in FP32)
    # and no grid past the cache takes another tile than these
    sizes = [12, 20, 33, 47, 64, 95, 127, 150, 200, 255, 350, 511, 767, 1000]
    large = [(a, b, c) for a in sizes for b in sizes for c in sizes if a * b * c > CACHED64]
    got = {}
    for q in range(0, len(large), 500):
        for kind, cached in ((0, CACHED64), (1, CACHED32)):
            for s, t in tiles(large[q:q + 500], kind).items():
                if np.prod(s, dtype=float) > cached:
                    got.setdefault(kind, set()).add(t[:2])
    assert got == {0: {(34, 14), (66, 10)}, 1: {(34, 14), (66, 10), (66, 14)}}


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FP64)
def test_fp64_sweeps_match_the_oracle(shape):
    g, o = _pair(_cfg(shape))
    g.begin_step(False)
    o.begin_step()
    g.refresh()
    o.refresh()
    for update, norms in ((True, False), (True, True), (True, False), (False, False), (False, True), (False, False)):
        g.iteration(update, norms)
        o.iteration(update, norms)
    _compare(g, o, STATE)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", FP32)
def test_fp32_sweeps_match_fp64_sweeps(shape):
    # 45 FP32 sweeps of a correction (the first from a stored residual, later
    # ones from two copies of the correction, checks and the last one storing
    # it) equal 45 linear FP64 sweeps to FP32 accuracy (rounding of 6e-8 per
    # sweep and value, a few per sweep, on the state's scale)
    from paper_2207_08716_amd import inputs, schedules
    cfg = _cfg(shape)
    f = inputs.initial_fields(cfg)
    a, b = schedules.make_grid(cfg, f), schedules.make_grid(cfg, f)
    for g in (a, b):
        g.begin_step(False)
        g.refresh(1.0, 1.0)
    a.solve_mixed(1e-300, 1e-30, 45, 1)
    for _ in range(45):
        b.iteration(False)
    for n in ("vx", "vy", "vz", "pt", "pf"):
        ref = b.get(n)
        assert np.abs(ref).max() > 0
        assert np.abs(a.get(n) - ref).max() <= 45 * 4 * 6e-8 * np.abs(ref).max(), n
