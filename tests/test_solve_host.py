"""The host side of the solves on a model of the device (solve_probe.hip): what
they leave in their stream when they return."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("solve") / "probe")
    # (host code alone, linked without the HIP runtime, whose calls the model answers)
    subprocess.run([HIPCC, "-x", "hip", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none",
                    "-no-hip-rt", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2207_08716_amd", "csrc"),
                    os.path.join(ROOT, "tests", "solve_probe.hip"), "-o", exe], check=True, capture_output=True)

    def go(scenario):
        out = subprocess.run([exe, scenario], check=True, capture_output=True, text=True, timeout=60).stdout
        return {k: float(v) for k, v in (line.split() for line in out.splitlines())}
    return go


@pytest.mark.parametrize("scenario", ["tail", "tail_static"])
def test_a_solve_at_its_limit_leaves_nothing_queued(run, scenario):
    # 15 sweeps to a check and 3 more: those read the gate, which in the
    # static scratch the next handle's solve writes over
    r = run(scenario)
    assert r["covers"] == 1 and r["status_a"] == 1 and r["iters_a"] == 18
    assert r["status_b"] == 0 and r["steps_b"] == r["iters_b"]
    assert r["queued_a"] == 0 and r["queued_b"] == 0
    assert r["steps_a"] == 18


def test_a_transposed_solve_at_its_limit_leaves_nothing_queued(run):
    r = run("tail_transposed")
    assert r["status"] == 1 and r["iters"] == 18 and r["steps"] == 18 and r["queued"] == 0


def test_a_mixed_solve_that_diverges_leaves_nothing_queued(run):
    r = run("mixed_nan")
    assert r["status"] == -3 and r["queued"] == 0


def test_the_static_solve_allocates_nothing(run):
    r = run("memory")
    assert r["mallocs_static"] == 0 and r["mallocs"] == 2
    assert r["status_static"] == r["status_linear"] == r["status_mixed"] == 0
    # and it is the other solve: 2^-(sweeps - 1) <= 1e-12 first holds at a check after 45
    assert r["iters_static"] == r["iters_linear"] == r["steps_static"] == r["steps_linear"] == 45
    assert r["rho_static"] == r["rho_linear"] and r["queued_static"] == 0


def test_a_solve_without_host_memory_is_the_same_solve(run):
    r, full = run("memory_refused"), run("memory")
    assert r.pop("mallocs") >= 2 and full.pop("mallocs") == 2 and r == full


def test_destroying_a_handle_waits_for_no_other_stream(run):
    # freeing pinned memory waits for the device: the block goes to the next
    # handle instead, up to a bound
    r = run("destroy")
    assert r["solved"] == 1 and r["solved_many"] == 1
    assert r["waited"] == 0 and r["mallocs_in_turn"] == 1
    assert r["kept"] <= 64
