"""The CG's control that host and device code share, checked on the CPU.

tests/host_control_driver.cpp includes the kernels' headers, is compiled for
the host only and runs one check per test; nothing here reaches a GPU.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not available")
    exe = str(tmp_path_factory.mktemp("control") / "host_control_driver")
    r = subprocess.run([hipcc, "--offload-host-only", "-O2", "-std=c++17", "-x", "hip",
                        os.path.join(HERE, "host_control_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


@pytest.mark.parametrize("check", ["loop_end_keeps_failure", "step_rounds_as_written", "strides_end"])
def test_control(driver, check):
    run = subprocess.run([driver, check], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
