"""The Python binding leaves the process's shared ctypes objects alone."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_import_leaves_pythonapi_as_it_is():
    code = ("import ctypes as C; f = C.pythonapi.PyBytes_FromStringAndSize; before = (f.restype, f.argtypes); "
            "from paper_1308_0653_amd import pdbm; assert (f.restype, f.argtypes) == before, f.restype; "
            "b = pdbm._new_bytes(None, 5); assert type(b) is bytes and len(b) == 5")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=60, cwd=ROOT)
    assert r.returncode == 0, r.stderr
