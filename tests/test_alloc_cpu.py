"""Failed device allocations in host code, with the HIP runtime's calls replaced by the test program's
(tests/sanitize/alloc_driver.cpp); no GPU needed."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2201_11655_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm toolchain missing")
def test_edge_index_allocation_failures(tmp_path):
    from paper_2201_11655_amd import vdmc
    vdmc.load()   # built
    exe = str(tmp_path / "alloc_driver")
    cmd = [CLANG, "-O1", "-g", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(ROCM, "include"), "-rdynamic",
           os.path.join(ROOT, "tests", "sanitize", "alloc_driver.cpp"), "-L" + PKG, "-l:libvdmc.so",
           "-L" + os.path.join(ROCM, "lib"), "-lamdhip64", "-Wl,-rpath," + PKG,
           "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-o", exe]
    r = subprocess.run(cmd, cwd=str(tmp_path), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], cwd=str(tmp_path), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "allocation failures ok" in r.stdout, r.stdout + r.stderr[-3000:]
