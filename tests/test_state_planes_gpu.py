"""The raw state in the caller's order: read_f, write_f and the checkpoint
blob hold the same values (the blob in the solve's precision), a state
written back or resumed at either buffer parity is bitwise the one saved and
steps on bitwise like it.  (That the velocity order is the oracle's is held
by the parity tests.)  Grids with padding columns, a whole strip, one column
and one row; float32 moves float64 planes in thirds."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [P.PDBM_FP64, P.PDBM_FP32])
@pytest.mark.parametrize("nr,nt,sector", [(20, 70, 8), (9, 64, 8), (33, 1, 8), (1, 17, 8), (12, 40, 3)])
def test_state_moves_bitwise_between_solvers(nr, nt, sector, precision):
    print(f"case {nr}x{nt} sector {sector} precision {precision}", flush=True)
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=0.3, dt=2e-6, r_split=0.6, p_noise=1e-3, seed=5)
    p, ic = P.make_params(**w.params_kw(), precision=precision), P.make_ic(**w.ic_kw())
    a = P.Solver(p, ic)
    a.step(3)
    f, lam = a.read_f()
    blob = a.get_state()
    real = np.float64 if precision == P.PDBM_FP64 else np.float32
    assert np.array_equal(np.frombuffer(blob, real, f.size, 32), f.ravel())
    assert np.array_equal(np.frombuffer(blob, np.float64, lam.size, 32 + f.size * real().itemsize), lam.ravel())
    b, c = P.Solver(p, None), P.Solver(p, None)
    b.set_state(blob)
    assert b.step_count == 3
    c.write_f(f, lam, step=4)  # the other buffer parity
    for s in (b, c):
        fs, ls = s.read_f()
        assert np.array_equal(fs, f) and np.array_equal(ls, lam)
    a.step(4)
    for s in (b, c):
        s.step(4)
        for x, y in zip(s.read_f(), a.read_f()):
            assert np.array_equal(x, y)


def test_writing_one_half_of_the_state_keeps_the_other():
    w = replace(W.small_fp64(), nr=10, ntheta=70, r_min=0.3, r_split=0.6, p_noise=1e-3, seed=6)
    s = P.Solver(P.make_params(**w.params_kw()), P.make_ic(**w.ic_kw()))
    f, lam = s.read_f()
    for step in (1, 2, 2, 5):  # to the other buffer, back, in place, to the other
        f = f + 1.0
        P._check(s.L.pdbm_write_f(s.h, P._dptr(f), None, step))
        assert all(np.array_equal(x, y) for x, y in zip(s.read_f(), (f, lam)))
    for step in (4, 4, 7):
        lam = lam + 0.5
        P._check(s.L.pdbm_write_f(s.h, None, P._dptr(lam), step))
        assert all(np.array_equal(x, y) for x, y in zip(s.read_f(), (f, lam)))


def test_drift_history_comes_whole_and_in_order():
    """4100 records wrap the ring of 4096; a shorter history does not."""
    w = replace(W.small_fp64(), nr=3, ntheta=1, r_min=0.3, dt=1e-6)
    s = P.Solver(P.make_params(**w.params_kw(), diag_every=1), P.make_ic(**w.ic_kw()))
    s.step(50)
    assert [r["step"] for r in s.diag_history()] == list(range(50))
    s.step(4050)
    assert [r["step"] for r in s.diag_history()] == list(range(4, 4100))
    assert [r["step"] for r in s.diag_history(cap=7)] == list(range(4093, 4100))
