"""A float32 solve's raw state in float64, through the device in pieces of as
many planes as the idle buffer holds (16 of whole strips, more of padded rows),
and for up to 2048 cells widened on the host: the values of the checkpoint, and
written back they give the same state."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nt,sector", [(32, 64, 8), (33, 64, 8), (70, 128, 8), (50, 70, 8), (400, 20, 3), (3000, 1, 8),
                                          (500, 5, 8)])
def test_float32_state_in_float64(nr, nt, sector):
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=0.3, dt=min(2e-6, 0.2 / nr / 12.5), r_split=0.6,
                p_noise=1e-3, seed=5)
    p, ic = P.make_params(**w.params_kw(), precision=P.PDBM_FP32), P.make_ic(**w.ic_kw())
    a, b = P.Solver(p, ic), P.Solver(p, None)
    a.step(3)
    f, lam = a.read_f()
    blob = a.get_state()
    assert np.isfinite(f).all()
    assert np.array_equal(np.frombuffer(blob, np.float32, f.size, 32), f.ravel().astype(np.float32))
    assert np.array_equal(f, f.astype(np.float32))
    assert np.array_equal(np.frombuffer(blob, np.float64, lam.size, 32 + 4 * f.size), lam.ravel())
    for step in (3, 4):  # into either buffer
        b.write_f(f, lam, step=step)
        for x, y in zip(b.read_f(), (f, lam)):
            assert np.array_equal(x, y)
    a.step(2)
    b.step(2)
    for x, y in zip(a.read_f(), b.read_f()):
        assert np.array_equal(x, y)
    a.close()
    b.close()
