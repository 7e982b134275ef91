"""The library's host code over a fake device (tests/host_stub.cpp): failures of a call half-way, and the parameters of the
launches, without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("no g++ or no HIP headers")
    exe = str(tmp_path_factory.mktemp("host_stub") / "host_stub")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-Wno-attributes", "-isystem", os.path.join(ROCM, "include"),
           "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host_stub.cpp"),
           os.path.join(ROOT, "paper_2505_18610_amd", "csrc", "kvq_host.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("scenario", ["batch_full_arena", "batch_failing_launch", "failed_block_is_refused", "mark_set_by_a_step",
                                      "mark_outlives_a_failing_step", "split_plans", "plans_follow_the_pages", "plans_follow_the_tier",
                                      "tile_costs_are_relative", "batch_shares", "batch_of_large_arenas", "sums_behind_a_failing_call"])
def test_host_code_over_a_fake_device(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
