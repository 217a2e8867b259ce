"""Every tile of the reactive sweep, on the smallest kinds of grids that the
rule sends to it: one plane per chunk, an even and an odd number of planes (the
two register sets alternate), ragged last tiles and chunks, cached and past the
last-level cache; plain and check sweeps, against the oracle."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle.reactive import ReactiveOracle
from paper_2207_08716_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FIELDS = ("xs", "pf", "phi", "dpfdt")

# grid: tile width, height, planes per chunk
GRIDS = {(18, 13, 11): (34, 4, 1), (11, 63, 15): (34, 6, 1), (9, 11, 165): (34, 6, 2), (8, 143, 10): (34, 10, 1),
         (15, 13, 167): (34, 10, 2), (9, 15, 280): (34, 10, 3), (13, 9, 204): (34, 14, 1), (7, 95, 53): (34, 14, 2),
         (44, 19, 175): (34, 14, 3), (34, 50, 129): (66, 10, 4), (121, 15, 175): (66, 10, 3),
         # past the cache (2.9 million cells)
         (132, 128, 174): (34, 14, 20), (143, 79, 258): (34, 14, 37), (107, 147, 198): (66, 10, 10),
         (104, 109, 277): (66, 10, 31)}
CACHED = 256e6 / 88      # cells


def test_the_grids_reach_every_tile(tmp_path):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "probe")
    subprocess.run([HIPCC, "-x", "hip", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none",
                    "-no-hip-rt", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2207_08716_amd", "csrc"),
                    os.path.join(ROOT, "tests", "pitch_probe.hip"), "-o", exe], check=True, capture_output=True)
    args = [str(v) for g in GRIDS for v in (*g, (g[0] + 32) // 32 * 32)]
    out = subprocess.run([exe, *args], check=True, capture_output=True, text=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert {r[:3]: r[5:8] for r in rows if r[4] == 4} == GRIDS
    tiles = {(w, h, nx * ny * nz <= CACHED) for (nx, ny, nz), (w, h, _) in GRIDS.items()}
    assert tiles == {(w, h, True) for w, h in ((34, 4), (34, 6), (34, 10), (34, 14), (66, 10))} | {
        (34, 14, False), (66, 10, False)}


@pytest.mark.gpu
@pytest.mark.parametrize("shape", GRIDS)
def test_sweeps_match_the_oracle_on_every_wave_tile(shape):
    from paper_2207_08716_amd.waves import Waves
    nx, ny, nz = shape
    rng = np.random.Generator(np.random.PCG64(nx * 1000 + nz))
    phi = 1e-2 * (1.0 + 1.5 * rng.random((nz, ny, nx)))
    ph = inputs.WavePhysics(lx=nx * 0.3, ly=ny * 0.3, lz=nz * 0.3)
    w, o = Waves(ph, nx, ny, nz, phi), ReactiveOracle(ph, nx, ny, nz, phi)
    w.begin_step()
    o.begin_step()
    w.iterate(13)          # pseudo steps before 1 and 11, a check after 10
    o.iterate(13)
    for n in FIELDS:
        ref = o.f[n]
        assert np.abs(w.get(n) - ref).max() <= 1e-12 * max(np.abs(ref).max(), 1e-300), n
    # a one-iteration change: each side within 1e-12 of the fields' scale
    scale = max(np.abs(o.f["phi"]).max(), np.abs(o.f["pf"]).max() / 10, np.abs(o.f["xs"]).max())
    assert abs(w.last_error() - o.last_err) <= 2e-12 * scale
