"""The pool of freed device blocks, on a stand-in for the HIP runtime (tests/native/pool.cpp): no block is
handed out while the device may still read it, and what is kept is bounded and can be given back."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2109_00170_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_pool(tmp_path):
    exe = str(tmp_path / "pool")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__", "-isystem", "/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "native", "pool.cpp"),
                           os.path.join(CSRC, "alcs_pack.cpp"), "-o", exe])
    out = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=120)
    assert out.returncode == 0 and b"pool OK" in out.stdout, out.stdout.decode(errors="replace")[-2000:]
