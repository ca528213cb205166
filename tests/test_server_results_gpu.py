"""A server reads the results of finished requests while the others step: each
equals its solo run's, whatever finishes beside it.  Results just below and
above the size from which their memory is in huge pages, and larger."""
import threading
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu

# 6 fields of 331 x 263 and 331 x 264 float64 lie on the two sides of 4 MiB
SHAPES = [(331, 263), (331, 264), (683, 256), (711, 253), (1100, 1013)]


def _made(nr, nt, seed=1, precision=P.PDBM_FP32, diag_every=0):
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, r_min=0.3, r_max=1.0, dt=2e-6, tau=5e-6, r_split=0.5513,
                p_noise=1e-3, seed=seed)
    return P.make_params(**w.params_kw(), precision=precision, diag_every=diag_every), P.make_ic(**w.ic_kw())


def test_server_results_read_beside_the_steps_of_others():
    """More requests than slots, which end at different chunks, some in the
    same one and the last alone; every result polled by two threads."""
    made = [_made(*SHAPES[i % len(SHAPES)], seed=i) for i in range(9)]
    counts = [4, 9, 9, 23, 4, 16, 0, 30, 41]
    srv = P.Server(hbm_cap_bytes=8 << 30, max_slots=4, chunk_steps=4)
    ids = [srv.submit(p, ic, n, keep_fields=True) for (p, ic), n in zip(made, counts)]
    peak = 0
    while not srv.wait(0.001):
        peak = max(peak, srv.stats()["running"])
    assert peak <= 4
    got = [[], []]

    def poll(k):
        for i in ids:
            got[k].append(srv.poll(i, fields=True))

    th = [threading.Thread(target=poll, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for (p, ic), n, a, b in zip(made, counts, *got):
        assert a[0] == P.PDBM_DONE and b[0] == P.PDBM_DONE
        s = P.Solver(p, ic)
        s.step(n)
        F, d = s.moments()
        assert np.array_equal(a[1], F) and np.array_equal(b[1], F)
        assert a[2]["step"] == n and a[2]["mass"] == b[2]["mass"] == d["mass"]
        s.close()
    for i in ids:
        srv.release(i)
    st = srv.stats()
    assert st["done"] == 9 and st["running"] == 0 and st["hbm_in_use"] == 0
    srv.close()
