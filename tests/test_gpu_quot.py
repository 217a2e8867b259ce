"""The kernels' quotient against the division, over the range that it states
and at its ends (quot_probe.hip, compiled and run here)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# units in the last place: a quotient corrected by its residual is less than
# one off; a residual rounded to the smallest subnormal adds at most half of one
RANGE, SMALL, SAME = 1, 2, 0
LIMITS = {"double_range": RANGE, "double_range_pair": RANGE, "double_range_low_end": RANGE, "double_range_high_end": RANGE,
          "double_small_dividends": SMALL, "double_field": RANGE, "double_specials": SAME, "double_pair_specials": SAME,
          "float_range": RANGE, "float_range_low_end": RANGE, "float_range_high_end": RANGE, "float_small_dividends": SMALL,
          "float_field": SAME, "float_field_subnormal": SAME, "float_specials": SAME, "float_field_specials": SAME}


def _build(exe):
    subprocess.run([HIPCC, "-x", "hip", *FLAGS, "-I", os.path.join(ROOT, "paper_2207_08716_amd", "csrc"),
                    os.path.join(ROOT, "tests", "quot_probe.hip"), "-o", exe], check=True, capture_output=True)


@pytest.mark.gpu
def test_quotient_over_its_range(tmp_path):
    exe = str(tmp_path / "probe")
    _build(exe)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = {name: int(worst) for name, worst, _ in (line.split() for line in r.stdout.splitlines())}
    assert got.keys() == LIMITS.keys()
    assert all(got[n] <= LIMITS[n] for n in got), (got, r.stderr)
