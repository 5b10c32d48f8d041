"""K splits summed inside a decode launch, seen from the host: the calls that
take that path, the arrival counters they get and the per-stream state, with
stand-ins for the HIP calls and the launchers (tests/native/host_arrive_driver.cpp).
CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_04031_amd", "csrc")


def test_arrival_counters(tmp_path):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers are not available")
    exe = tmp_path / "drv"
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(ROOT, "tests", "native", "host_arrive_driver.cpp"),
           os.path.join(CSRC, "tl_api.cpp"), os.path.join(CSRC, "tl_read_amp.cpp"), os.path.join(CSRC, "tl_view.cpp"),
           "-o", str(exe)]
    out = subprocess.run(cmd, capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-3000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"), timeout=300)
    assert run.returncode == 0, (run.stdout + run.stderr)[-3000:]
