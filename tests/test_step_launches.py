"""The launches pdbm_step makes of single solves, from the library's host code
on a model of the GPU (tests/host/launch_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_of_single_solves(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_1308_0653_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "launch_check.cpp"), "-o", exe, "-lpthread"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "launches ok" in r.stdout, r.stderr[-3000:]
