"""Wide rows: the sweeps address a tile's rows in a plane with 32 bits, so the
tile rules take lower tiles where the row pitch asks for it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("pitch") / "probe")
    subprocess.run([HIPCC, "-x", "hip", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none",
                    "-no-hip-rt", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2207_08716_amd", "csrc"),
                    os.path.join(ROOT, "tests", "pitch_probe.hip"), "-o", exe], check=True, capture_output=True)
    shapes = [(nx, ny, nz, p) for nx in (40, 1000, 19_000_000) for ny in (2, 3, 8, 40, 500) for nz in (2, 9, 200)
              for p in (19_173_952, 19_173_984, 26_843_584, 38_347_936, 44_739_264, 67_108_832)]
    out = subprocess.run([exe, *[str(v) for s in shapes for v in s]], check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_every_pitch_up_to_67_million_has_a_tile(rows):
    for nx, ny, nz, pitch, kind, w, h, kz, elem, taken in rows:
        assert w in (66, 34) and kz >= 1, (nx, ny, nz, pitch, kind)
        # a tile holds its own rows of the box, at most all of them
        assert min(h, ny + 1) * pitch * elem <= 0x7fffffff, (nx, ny, nz, pitch, kind, w, h)
        assert taken in ((-1,) if kind < 4 else (1,)), (nx, ny, nz, pitch, kind, w, h)
