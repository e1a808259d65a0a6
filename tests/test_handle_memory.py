"""Handles when device memory runs out, and their tuning by summation mode (no GPU).

The library's host side is compiled as it is, without its kernels, and linked with a stand-in for the HIP runtime whose
device memory has a budget.  A build that cannot get its buffers leaves a handle that every call refuses (ESTATE)
until a build succeeds; the force pass takes the least lists where the wanted ones do not fit.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2110_11398_amd", "csrc")
OK, EINVAL, ENOMEM, ESTATE = 0, -1, -2, -6


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("handle")
    exe = str(d / "handle")
    inc = ["-I", os.path.join(os.path.dirname(HERE), "include")]
    for src, obj in ((os.path.join(CSRC, "api.hip"), "api.o"), (os.path.join(HERE, "handle_main.cpp"), "main.o")):
        r = subprocess.run([hipcc, "-O1", "-w", "-std=c++17", "-x", "hip", "--offload-host-only", *inc, "-c", src, "-o",
                            str(d / obj)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([hipcc, "-o", exe, str(d / "api.o"), str(d / "main.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return subprocess.run([exe], capture_output=True, text=True, check=True).stdout.splitlines()


def test_a_built_handle_serves_every_call(lines):
    assert lines[0] == f"build {OK}"
    assert lines[1].split()[1:] == [str(OK)] * 13 + ["null=0"]


def test_a_failed_build_leaves_a_handle_that_every_call_refuses(lines):
    assert lines[3] == f"grow {ENOMEM}"
    assert lines[4].split()[1:] == [str(ESTATE)] * 13 + ["null=0"]
    assert lines[5] == f"build {OK}"


def test_the_force_pass_takes_the_least_lists_where_memory_is_short(lines):
    want, least = lines[9].split()[1], lines[9].split()[3]
    assert lines[6] == f"build {OK} forces {OK} slots {want} short 1 again {OK} null=0"
    assert lines[7] == f"build {OK} forces {OK} slots {least} short 1 again {OK} null=0"
    assert lines[8] == f"build {OK} forces {ENOMEM} again {OK} null=0"


def test_fp64_sums_and_few_lanes_take_two_sinks_per_lane_unless_set(lines):
    assert lines[10:14] == ["sinks 4 4 2 get 4", "sinks 4 4 4 get 4", "sinks 1 1 1 get 1", "sinks 4 4 2 get 4"]
    assert lines[14] == "sinks 2 2 2 get 4"


def test_smaller_calls_on_a_handle_allocate_nothing(lines):
    got = lines[15:]
    assert got[0].startswith(f"boxes 8 rc {OK} ")
    assert got[1:] == [f"boxes {b} rc {OK} allocations 0" for b in (4, 2, 1, 3, 8, 4, 2, 1, 3)]
