"""Wavefronts of a workgroup that march strips side by side hand the ends of
their rows on to each other; where a row of strips begins and ends within the
workgroup follows from the number of strips and, in a pack, from the members
before.  Every field is bitwise the same wherever that is: alone, and behind a
first member of one to three strips that shifts the workgroups' borders.  One
to nine strips, closed around the circle on whole strips and not, one octant
to eight, the disc, blocks of 2 rows and more."""
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = [(150, 192, 8), (90, 256, 4), (140, 258, 8), (75, 320, 5), (66, 384, 3), (52, 400, 1), (130, 512, 8),
         (47, 576, 2), (33, 500, 7)]


def _made(nr, nt, sector, precision, seed=2, disc=False):
    w = replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=0.0 if disc else 0.3, r_max=1.0, dt=1e-6,
                tau=5e-6, r_split=0.5513, p_noise=1e-3, seed=seed)
    flags = P.PDBM_ALLOW_CFL if disc else 0
    return P.make_params(**w.params_kw(), precision=precision, flags=flags), P.make_ic(**w.ic_kw())


@pytest.mark.parametrize("precision", [P.PDBM_FP64, P.PDBM_FP32])
@pytest.mark.parametrize("first", [(2, 64), (2, 128), (2, 192), (17, 64)])
def test_fields_do_not_depend_on_the_workgroups_borders(first, precision):
    made = [_made(*g, precision) for g in GRIDS] + [_made(30, 40 * 4, 4, precision, disc=True)]
    got = {}
    for lead in (False, True):
        ms = ([_made(*first, 1, precision)] if lead else []) + made
        b = P.Batch([m[0] for m in ms], [m[1] for m in ms], chunk_steps=5)
        b.step(11)
        got[lead] = [b.moments(i, check=False)[0] for i in range(len(ms))][lead:]
        b.close()
    for k, m in enumerate(made):
        s = P.Solver(*m)
        s.step(11)
        F, _ = s.moments(check=False)
        assert np.isfinite(F).all(), k
        assert np.array_equal(F, got[False][k]) and np.array_equal(F, got[True][k]), (k, GRIDS[k:k + 1])
        s.close()
