"""The steps' host side over a stand-in for the HIP runtime (tests/host_steps.cpp), compiled for the CPU: what no GPU run can show at will
(a refused call's allocations, a launch that fails, queue depths, a stream under capture)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_19867_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the HIP headers")
    out = str(tmp_path_factory.mktemp("host") / "host_steps")
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                            "-I", CSRC, *[os.path.join(CSRC, f) for f in ("ctx.cpp", "steps.cpp", "pool.cpp", "rope.cpp")],
                            os.path.join(ROOT, "tests", "host_steps.cpp"), "-o", out, "-lpthread"], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    return out


@pytest.mark.parametrize("scenario", ["refused_copies", "failed_launch", "captured", "captured_prefill", "parts", "staged", "in_flight", "merges", "launches", "devices", "shares", "dense_rows"])
def test_host_side(exe, scenario):
    run = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout == "ok\n", run.stderr[-2000:]
