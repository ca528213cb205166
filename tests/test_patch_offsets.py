"""Every buffer and LDS access of the patch kernel, and the accesses of marched
strips with mixed octants, inside their buffers: checked on the host from the
header the kernels use (tests/host/patch_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_patch_accesses_in_bounds(tmp_path):
    exe = str(tmp_path / "patch_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_1308_0653_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "patch_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=110)
    print(r.stdout)
    assert r.returncode == 0 and " 0 failed" in r.stdout, r.stderr[-3000:]
