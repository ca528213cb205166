"""The Python binding leaves the process's shared ctypes objects alone and takes
a checkpoint as bytes only."""
import os
import subprocess
import sys
from types import SimpleNamespace

import pytest

from paper_1308_0653_amd import pdbm as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_import_leaves_pythonapi_as_it_is():
    code = ("import ctypes as C; f = C.pythonapi.PyBytes_FromStringAndSize; before = (f.restype, f.argtypes); "
            "from paper_1308_0653_amd import pdbm; assert (f.restype, f.argtypes) == before, f.restype; "
            "b = pdbm._new_bytes(None, 5); assert type(b) is bytes and len(b) == 5")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=60, cwd=ROOT)
    assert r.returncode == 0, r.stderr


def test_set_state_takes_bytes_only():
    """An int is a count to bytes(), and a bytearray may change: neither is a
    checkpoint."""
    s = P.Solver.__new__(P.Solver)
    s.h, got = None, []
    s.L = SimpleNamespace(pdbm_set_state=lambda h, blob, n: got.append((blob.value[:n], n)) or P.PDBM_OK)
    s.set_state(b"abc")
    assert got == [(b"abc", 3)]
    for bad in (5, bytearray(b"abc"), memoryview(b"abc"), [1, 2], "abc", None):
        with pytest.raises(TypeError):
            s.set_state(bad)
    assert len(got) == 1
