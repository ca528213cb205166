"""A pack chooses the length of its members' row blocks anew with every change
of its members.  It doesn't show in a result: every cell's update is rounded
the same way in any block, so a member's fields equal its solo run's bitwise."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu


def _params(nr, nt, seed, precision, diag_every):
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, r_min=0.3, r_max=1.0, dt=2e-6, tau=5e-6, r_split=0.5513,
                p_noise=1e-3, seed=seed)
    return P.make_params(**w.params_kw(), precision=precision, diag_every=diag_every), P.make_ic(**w.ic_kw())


# one member to many: blocks of 2 rows, some length between, 16 rows; drift
# records keep the blocks at 16 rows
@pytest.mark.parametrize("precision", [P.PDBM_FP64, P.PDBM_FP32])
@pytest.mark.parametrize("members,diag_every", [(1, 0), (1, 1), (3, 0), (9, 0), (9, 10), (40, 0)])
def test_packs_of_any_size_equal_solo_runs_bitwise(members, diag_every, precision):
    shapes = [(300 - 7 * (i % 5), 200 + 63 * (i % 4)) for i in range(members)]
    made = [_params(nr, nt, i, precision, diag_every) for i, (nr, nt) in enumerate(shapes)]
    b = P.Batch([m[0] for m in made], [m[1] for m in made], chunk_steps=6)
    b.step(15)
    for i in {0, members // 2, members - 1}:
        s = P.Solver(*made[i])
        s.step(15)
        F, _ = s.moments()
        Fb, _ = b.moments(i)
        assert np.array_equal(F, Fb), (i, shapes[i], np.abs(F - Fb).max())
        s.close()
    b.close()


# more wavefronts than the device holds at once: 9 and 10 rows alone, 16 in a pack that makes drift records
@pytest.mark.parametrize("nr,nt,precision", [(1100, 1024, P.PDBM_FP64), (2400, 1024, P.PDBM_FP32)])
def test_single_solves_beyond_one_round_equal_blocks_of_16_rows_bitwise(nr, nt, precision):
    p, ic = _params(nr, nt, 4, precision, 1)
    s = P.Solver(p, ic)
    s.step(7)
    b = P.Batch([p], [ic], chunk_steps=4)
    b.step(7)
    F, _ = s.moments()
    assert np.array_equal(F, b.moments(0)[0])
    hist = s.diag_history()
    assert [r["step"] for r in hist] == list(range(7))
    # the record of step k is that of the state k steps in (the same 1e6 or more terms, added up in another order)
    t = P.Solver(p, ic)
    t.step(6)
    d = t.moments()[1]
    assert abs(hist[6]["mass"] - d["mass"]) <= 1e-11 * d["mass"] and hist[6]["n_nonfinite"] == 0
    assert abs(hist[6]["energy"] - d["energy"]) <= 1e-11 * abs(d["energy"])
    t.close()
    s.close()
    b.close()
