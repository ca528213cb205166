"""A cell's new state does not depend on the kernel, the strip, the row block
or the patch it is computed in: every kernel rounds the update the same way.
Each case is run by the launches chosen for it, by other row blocks
(PDBM_ROWS_PER_WAVE) and one step at a time (PDBM_FUSE=0, odd and even step
counts), the environment being read once per process, and every value of f
and lambda must come out bitwise equal.  The grids: octants that are whole
strips, cut by strips and narrower than one, periodic images past the last
column, sectors, a disc, fewer columns than octants, single columns, and one
grid for each shape of patch."""
import os
import subprocess
import sys
from dataclasses import replace

import numpy as np
import pytest

from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GRIDS = [(37, 512, 8), (20, 200, 8), (21, 65, 8), (9, 20, 8), (18, 8, 8), (11, 5, 8), (3, 2, 8), (24, 130, 3),
         (12, 64, 1), (17, 128, 2), (40, 1, 8), (33, 1, 1), (500, 1, 2), (64, 64, 8), (100, 100, 8), (200, 180, 8),
         (300, 130, 8)]
DISCS = [(14, 40, 4), (19, 24, 1), (10, 3, 4)]
VARIANTS = [{}, {"PDBM_ROWS_PER_WAVE": "3"}, {"PDBM_ROWS_PER_WAVE": "16"}, {"PDBM_FUSE": "0"}]


def run_all():
    out = {}
    for nr, nt, sector in GRIDS + DISCS:
        disc = (nr, nt, sector) in DISCS
        w = replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=0.0 if disc else 0.3, r_max=1.0, dt=2e-6,
                    tau=5e-6, r_split=0.5513, p_noise=1e-3, seed=nr)
        for prec in (P.PDBM_FP64, P.PDBM_FP32):
            for tau in (False, True):
                flags = (P.PDBM_TAU_FIELD if tau else 0) | (P.PDBM_ALLOW_CFL if disc else 0)
                s = P.Solver(P.make_params(**w.params_kw(), precision=prec, flags=flags, diag_every=3),
                             P.make_ic(**w.ic_kw()))
                if tau:
                    s.set_tau(np.random.default_rng(1).uniform(3e-6, 3e-5, (nr, nt)))
                for n in (5, 2, 8):
                    s.step(n)
                f, lam = s.read_f()
                key = f"{nr}x{nt}s{sector}p{prec}t{int(tau)}{'d' if disc else ''}"
                assert np.isfinite(f).all(), key
                out[key], out[key + "l"] = f, lam
                s.close()
    return out


CHILD = """
import sys
import numpy as np
sys.path.insert(0, {root!r})
from tests.test_bitwise_paths_gpu import run_all
np.savez({out!r}, **run_all())
print("child done", flush=True)
"""


def _child(tmp_path, k, env):
    out = str(tmp_path / f"v{k}.npz")
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT, out=out)], env=dict(os.environ, **env), cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return dict(np.load(out))


def test_every_launch_form_gives_the_same_bits(tmp_path):
    ref = _child(tmp_path, 0, VARIANTS[0])
    for k, env in enumerate(VARIANTS[1:], 1):
        print("variant", env, flush=True)
        got = _child(tmp_path, k, env)
        bad = [key for key in ref if not np.array_equal(ref[key], got[key])]
        assert not bad, (env, bad)
