"""The request server's host code on a model of the GPU (tests/host/
server_check.cpp): a finished request is done while the next chunk of the
others is in flight; its slot and its memory serve the next request at once;
and no use of it from several threads races, hangs or leaks, whenever it is
destroyed (also under ThreadSanitizer)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"  # (its ThreadSanitizer knows timed waits on the steady clock)


def _build(out, compiler, *extra):
    subprocess.run([compiler, "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_1308_0653_amd", "csrc"), *extra,
                    os.path.join(ROOT, "tests", "host", "server_check.cpp"), "-o", out, "-lpthread"],
                   check=True, capture_output=True, text=True)
    return out


def _run(exe, *args):
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=110)
    print(r.stdout)
    assert r.returncode == 0 and f"server {args[0]} ok" in r.stdout, (r.stdout + r.stderr)[-3000:]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("server") / "check"), "g++")


@pytest.mark.parametrize("what", ["slots", "memory", "reports", "fields"])
def test_finished_requests_leave_at_once(exe, what):
    _run(exe, what)


def test_server_under_thread_sanitizer(tmp_path):
    if not os.path.exists(CLANG):
        pytest.skip("no ROCm toolchain")
    tsan = _build(str(tmp_path / "check_tsan"), CLANG, "-fsanitize=thread")
    for what in ("slots", "reports", "fields"):
        _run(tsan, what)
    _run(tsan, "random", "1", "100")
