"""The host's rules for launches (csrc/adagc_internal.h) on the CPU, compiled into small drivers with the HIP runtime's headers but without
the runtime."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="needs g++ and the HIP headers")


def _driver(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2502_11034_amd", "csrc"), "-isystem", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", name + ".cpp"), "-o", exe], check=True)
    return exe


def test_a_stream_that_cannot_be_asked_leaves_no_error_behind(tmp_path):
    """The NULL stream while another stream is captured: the question fails, the step's launches must not report that."""
    res = subprocess.run([_driver(tmp_path, "issues_now_check")], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
