"""What the C ABI's host logic enqueues, and which storage form it names for the
buffers read, with the kernel launchers replaced by ones that write lines
(tests/abi_driver/host_forms_check.cpp); no GPU."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = os.path.join(ROOT, "tests", "abi_driver")
CSRC = os.path.join(ROOT, "paper_1703_00186_amd", "csrc")


def test_launches_and_their_forms(tmp_path):
    if not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "host_forms_check")
    cmd = ["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(CSRC, "lb_api.hip"),
           os.path.join(DRIVER, "host_forms_check.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    assert r.returncode == 0, r.stdout + r.stderr
