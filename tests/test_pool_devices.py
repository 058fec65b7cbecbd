"""The device buffer pool on two devices, against a stand-in for the HIP runtime
(a host program): a release waits for the stream of the buffers' device."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_release_waits_on_the_buffers_device(tmp_path):
    cxx = shutil.which("clang++", path=os.path.join(ROCM, "llvm", "bin")) or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no clang++ (the sources use _Float16 in declarations)")
    exe = str(tmp_path / "pool_devices")
    csrc = os.path.join(ROOT, "paper_2303_05455_amd", "csrc")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", csrc, "-x", "c++", os.path.join(csrc, "pool.hip"),
                    os.path.join(HERE, "pool_devices.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
