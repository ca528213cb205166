"""Grids of fewer columns than octants, which are stepped on patches: a solve
without allocation takes as many rows as with 16 rows to a wavefront, and the
tall patches of many rows with drift records step like the others."""
import ctypes as C
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W


def _made(nr, nt, precision, diag_every, sector=8):
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=0.3, r_max=1.0, dt=0.25 / nr / 12.5,
                tau=0.5 / nr / 12.5, r_split=0.5513, p_noise=1e-3, seed=nt)
    return P.make_params(**w.params_kw(), precision=precision, diag_every=diag_every), P.make_ic(**w.ic_kw())


# 64 records x wavefronts x 40 bytes and the rest fit the static scratch of
# 16 MiB up to about 6400 wavefronts, 102 thousand rows
@pytest.mark.parametrize("precision", [P.PDBM_FP64, P.PDBM_FP32])
@pytest.mark.parametrize("diag_every", [0, 1])
def test_noalloc_takes_narrow_grids_of_many_rows(diag_every, precision):
    n, h = C.c_size_t(0), C.c_void_p()

    def refused(nr, nt, sector):
        p, _ = _made(nr, nt, precision, diag_every, sector)
        # a state buffer of 0 bytes is refused too, but only after the scratch
        rc = P.lib().pdbm_create_noalloc(C.byref(p), None, C.c_void_p(1 << 20), C.byref(n), None, C.byref(h))
        assert rc != P.PDBM_OK and not h.value
        return b"static scratch" in P.lib().pdbm_last_error()

    for nr, nt, sector in [(100, 7, 8), (5121, 7, 8), (40000, 6, 8), (40000, 7, 8), (60000, 5, 8), (80000, 4, 8),
                           (80000, 4, 5), (100000, 2, 8), (100000, 7, 8), (100000, 2, 3)]:
        assert not refused(nr, nt, sector), (nr, nt, sector)
    for nt in (2, 5, 7):
        assert refused(110000, nt, 8), nt


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [P.PDBM_FP64, P.PDBM_FP32])
def test_tall_patches_step_like_the_others_bitwise(precision):
    """5121 and 5200 rows of 7 and 5121 of 6 columns, just over and well under
    1024 patches: with drift records on tall patches, without on the others,
    alone and both in one pack.  The records are those of the states."""
    shapes = [(5121, 7), (5200, 7), (5121, 6), (31, 7)]
    plain = [_made(nr, nt, precision, 0) for nr, nt in shapes]
    recs = [_made(nr, nt, precision, 1) for nr, nt in shapes]
    ms = [m for pair in zip(plain, recs) for m in pair]
    b = P.Batch([m[0] for m in ms], [m[1] for m in ms], chunk_steps=5)
    b.step(7)
    for k, (nr, nt) in enumerate(shapes):
        print(f"{nr}x{nt}", flush=True)
        a, r = P.Solver(*plain[k]), P.Solver(*recs[k])
        r.step(6)
        before = r.moments()[1]
        r.step(1)
        a.step(7)
        F = a.moments()[0]
        assert np.isfinite(F).all()
        for x, y in zip(a.read_f(), r.read_f()):
            assert np.array_equal(x, y)
        for i in (2 * k, 2 * k + 1):
            assert np.array_equal(F, b.moments(i)[0])
        h = r.diag_history()
        assert [d["step"] for d in h] == list(range(7))
        assert h[6]["n_nonfinite"] == h[6]["n_nonphys"] == 0
        # the same terms, up to 36400 of one sign, added up in another order
        for q in ("mass", "energy"):
            assert abs(h[6][q] - before[q]) <= 1e-11 * abs(before[q])
        a.close()
        r.close()
    b.close()


@pytest.mark.gpu
@pytest.mark.parametrize("diag_every", [0, 2])
@pytest.mark.parametrize("nr,nt,sector", [(1000, 1, 8), (64, 2, 2), (64, 8, 8), (200, 20, 8), (400, 7, 8), (64, 64, 8)])
def test_a_cap_of_the_solves_own_bytes_admits_it(nr, nt, sector, diag_every):
    """A packed solve takes no more memory than alone (pdbm_state_bytes)."""
    p, ic = _made(nr, nt, P.PDBM_FP64, diag_every, sector)
    srv = P.Server(hbm_cap_bytes=P.pdbm_state_bytes(p), max_slots=1, chunk_steps=4)
    rid = srv.submit(p, ic, 4)
    assert srv.wait(30.0) and srv.poll(rid)[0] == P.PDBM_DONE
    srv.close()
