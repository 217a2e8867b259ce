"""The sweeps' tile rule, compiled host-only from the library's header: every
grid gets a tile the kernels are built for, whose chunks cover it, and a
number of blocks that the norms' scratch holds; the choices the measurements
rest on."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
F64, F32, NORM64, NORM32 = range(4)
BUILT = {F64: {(66, 10), (66, 6), (34, 14), (34, 6), (34, 4)}, F32: {(66, 14), (66, 10), (66, 6), (34, 14), (34, 6)},
         NORM64: {(66, 7), (34, 14), (34, 6), (34, 4)}, NORM32: {(66, 7), (34, 14), (34, 6), (34, 4)}}
SIZES = [2, 3, 5, 8, 16, 31, 33, 40, 64, 66, 95, 127, 129, 200, 255, 511, 767, 1100]


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("tiling") / "probe")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2207_08716_amd", "csrc"),
                    os.path.join(ROOT, "tests", "tiling_probe.hip"), "-o", exe], check=True, capture_output=True)
    shapes = [(a, b, c) for a in SIZES for b in SIZES[::2] for c in SIZES[::3]] + [(n, n, n) for n in SIZES]
    out = subprocess.run([exe, *[str(v) for s in shapes for v in s]], check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, l.split())) for l in out.splitlines()]


def test_every_grid_gets_a_built_tile_that_covers_it(rows):
    for nx, ny, nz, kind, w, h, kz, blocks, old, most in rows:
        assert (w, h) in BUILT[kind], (nx, ny, nz, kind, w, h)
        assert 1 <= kz <= 256
        tiles = -(-nx // (w - 2)) * -(-ny // (h - 2))
        assert blocks == tiles * -(-nz // kz) and blocks >= 1
        # per-block maxima: no grid needs more scratch than the tile of 66 x 7
        # threads on power-of-two chunks, or than 4096 blocks
        assert most <= max(4096, old), (nx, ny, nz, most, old)


def test_choices_the_measurements_rest_on(rows):
    got = {r[:4]: r[4:7] for r in rows}
    assert got[(511, 511, 511, F64)] == (66, 10, 256)
    assert got[(127, 127, 127, F64)] == (66, 10, 16)
    assert got[(95, 95, 95, F64)] == (34, 14, 10)
    assert got[(64, 64, 64, F64)] == (66, 10, 2)
    assert got[(16, 16, 16, F64)] == (34, 4, 1)
    assert got[(95, 95, 95, F32)] == (34, 14, 3)
    assert got[(127, 127, 127, F32)] == (66, 10, 8)
