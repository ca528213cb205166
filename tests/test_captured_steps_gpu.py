"""pdbm_step captured in a HIP graph: a call of 4 steps (16 for a single theta
column) finds the state where it left it, so that every replay takes as many
steps on, on patches as on marching wavefronts.  Replays with eager work of the
program between them, each checked against eager steps bitwise."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu


# patches of 4, 3 and 2 steps per launch, narrow ones, columns of 24 steps, of
# 8 (marched) and at a disc centre, and marched strips
@pytest.mark.parametrize("precision", [P.PDBM_FP64, P.PDBM_FP32])
@pytest.mark.parametrize("nr,nt,sector,r_min,steps", [
    (64, 64, 8, 0.3, 4), (100, 100, 8, 0.3, 4), (100, 100, 8, 0.3, 12), (300, 130, 8, 0.3, 8), (300, 200, 8, 0.3, 4),
    (30, 5, 8, 0.3, 4), (500, 1, 8, 0.3, 16), (500, 1, 2, 0.0, 48), (41000, 1, 8, 0.3, 16), (200, 700, 8, 0.3, 4)])
def test_captured_steps_replay(nr, nt, sector, r_min, steps, precision):
    torch = pytest.importorskip("torch")
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=r_min, r_max=1.0, dt=min(2e-6, 0.25 / nr / 12.5),
                tau=5e-6, r_split=0.5513, p_noise=1e-3, seed=nr)
    p = P.make_params(**w.params_kw(), precision=precision, flags=P.PDBM_ALLOW_CFL if r_min == 0.0 else 0)
    ic = P.make_ic(**w.ic_kw())
    st = torch.cuda.Stream()
    s, e = P.Solver(p, ic, stream=st), P.Solver(p, ic, stream=st)
    s.step(steps)  # (loads the kernels)
    e.step(steps)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        s.step(steps)
    other = torch.zeros(1000, device="cuda")
    for k in range(3):
        with torch.cuda.stream(st):
            g.replay()
        other += 1.0
        torch.cuda.synchronize()
        e.step(steps)
        for x, y in zip(s.read_f(), e.read_f()):
            assert np.isfinite(y).all() and np.array_equal(x, y), k
    s.close()
    e.close()
