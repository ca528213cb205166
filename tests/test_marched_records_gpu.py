"""The two-step kernel's drift records, checkpoints and restores on grids that
would be stepped on patches otherwise: in a child process with row blocks of 3
and of 16 rows, where every solve of two columns or more is marched.

- Every record, of both steps of a pair and of single steps, is that of a
  process whose launches take single steps (PDBM_FUSE=0): counts exactly, sums
  but for the order in which N terms are added, within 2 N 2^-53 of the sum of
  their magnitudes (the states are equal bitwise).
- In float64 it is also the oracle's, within the bound of the fields, 1e-10.
- A state saved after an odd number of pairs, or restored at an odd step, goes
  on bitwise as it would have."""
import os
import subprocess
import sys
from dataclasses import replace

import numpy as np
import pytest

from oracle import oracle as O
from paper_1308_0653_amd import pdbm as P
from paper_1308_0653_amd import workloads as W

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SUMS = ("mass", "energy", "chem")

# nr, ntheta, sector, disc, diag_every, steps: image lanes past the last
# column and none, one strip to four, rows that end a block and not, octants
# that are whole strips and cut by them, sectors, discs with whole octants
CASES = [(33, 130, 8, False, 1, 130), (20, 70, 8, False, 3, 61), (40, 64, 8, False, 1, 9), (17, 200, 8, False, 2, 13),
         (37, 512, 8, False, 1, 6), (21, 130, 3, False, 1, 11), (16, 64, 1, False, 1, 8), (19, 128, 2, True, 1, 9),
         (34, 256, 4, True, 1, 8), (14, 40, 4, True, 3, 10), (1, 65, 8, False, 1, 7), (2, 64, 8, False, 1, 4)]


def _workload(nr, nt, sector, disc, seed=3):
    return replace(W.small_fp64(), nr=nr, ntheta=nt, sector=sector, r_min=0.0 if disc else 0.3, r_max=1.0, dt=2e-6,
                   tau=5e-6, r_split=0.5513, p_noise=1e-3, seed=seed)


def _solver(w, precision, diag_every):
    flags = P.PDBM_ALLOW_CFL if w.r_min == 0.0 else 0
    return P.Solver(P.make_params(**w.params_kw(), precision=precision, diag_every=diag_every, flags=flags),
                    P.make_ic(**w.ic_kw()))


def _history(s):
    return np.array([[h["step"], h["n_nonfinite"], h["n_nonphys"], *(h[k] for k in SUMS)] for h in s.diag_history()])


def _planted(f):
    """One cell of NaN, one with every f negated (rho < 0, T unchanged), in
    lanes and rows inside their strips and blocks."""
    f[:, 10, 30] = np.nan
    f[:, 30, 100] *= -1.0


def run_all():
    out = {}
    for prec in (P.PDBM_FP64, P.PDBM_FP32):
        for c in CASES:
            nr, nt, sector, disc, every, n = c
            print("case", c, prec, flush=True)
            s = _solver(_workload(nr, nt, sector, disc), prec, every)
            s.step(n)
            key = f"{nr}x{nt}s{sector}p{prec}"
            out[key] = _history(s)
            out[key + "f"], out[key + "l"] = s.read_f()
            s.close()
        # bad cells, over a pair and an odd step
        s = _solver(_workload(40, 130, 8, False), prec, 1)
        f, lam = s.read_f()
        _planted(f)
        s.write_f(f, lam)
        s.step(3)
        out[f"badp{prec}"] = _history(s)
        s.close()
        # saved after three pairs, restored into another solve; and restored at an odd step
        w = _workload(24, 130, 8, False)
        a, b, c = (_solver(w, prec, 1) for _ in range(3))
        a.step(6)
        b.set_state(a.get_state())
        c.step(1)
        for _ in range(6):
            c.step(1)
        a.step(1)
        b.step(1)
        assert np.array_equal(a.noneq(), c.noneq())
        b.set_state(c.get_state())  # step 7
        for s in (a, b, c):
            s.step(5)
            assert s.step_count == 12
        for s in (b, c):
            for x, y in zip(s.read_f(), a.read_f()):
                assert np.array_equal(x, y)
        out[f"oddp{prec}"] = _history(b)
        for s in (a, b, c):
            s.close()
    return out


CHILD = """
import sys
import numpy as np
sys.path.insert(0, {root!r})
from tests.test_marched_records_gpu import run_all
np.savez({out!r}, **run_all())
print("child done", flush=True)
"""


def _child(path, env):
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT, out=path)], env=dict(os.environ, **env), cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return dict(np.load(path))


def _check(got, want, terms, key):
    """Rows of (step, counts, sums): the same but for the order of summation."""
    assert np.array_equal(got[:, :3], want[:, :3]), key
    bound = 2 * terms * 2.0**-53
    for i, k in enumerate(SUMS, 3):
        # (one negated cell of many: the magnitudes add up to less than twice the sum)
        assert (np.abs(got[:, i] - want[:, i]) <= 2 * bound * np.abs(want[:, i])).all(), (key, k)


@pytest.fixture(scope="module")
def single(tmp_path_factory):
    return _child(str(tmp_path_factory.mktemp("records") / "single.npz"), {"PDBM_FUSE": "0"})


@pytest.mark.parametrize("rows", ["3", "16"])
def test_pairs_make_the_records_of_single_steps_and_of_the_oracle(single, rows, tmp_path):
    got = _child(str(tmp_path / "pairs.npz"), {"PDBM_ROWS_PER_WAVE": rows})
    assert set(got) == set(single)
    for prec in (P.PDBM_FP64, P.PDBM_FP32):
        for c in CASES:
            nr, nt, sector, disc, every, n = c
            key = f"{nr}x{nt}s{sector}p{prec}"
            assert list(got[key][:, 0]) == list(range(0, n, every)), key
            assert not got[key][:, 1:3].any(), key
            _check(got[key], single[key], nr * nt, key)
            assert np.array_equal(got[key + "f"], single[key + "f"]) and np.array_equal(got[key + "l"], single[key + "l"])
        bad = got[f"badp{prec}"]
        # (the bad cell spreads to its four neighbours in each step)
        assert list(bad[:2, 1]) == [1, 5] and bad[0, 2] == 1 and np.isfinite(bad).all()
        _check(bad, single[f"badp{prec}"], 40 * 130, f"bad {prec}")
        odd = got[f"oddp{prec}"]
        assert list(odd[:, 0]) == list(range(7, 12))
        _check(odd, single[f"oddp{prec}"], 24 * 130, f"odd {prec}")
    for c in CASES:
        nr, nt, sector, disc, every, n = c
        w = _workload(nr, nt, sector, disc)
        o = O.Solver(O.make_params(**w.params_kw()))
        o.init_ic(**w.ic_kw())
        for row in got[f"{nr}x{nt}s{sector}p{P.PDBM_FP64}"]:
            o.step(int(row[0]) - o.step_count)
            ref = o.diag()
            for i, k in enumerate(SUMS, 3):
                assert abs(row[i] - ref[k]) <= 1e-10 * abs(ref[k]), (c, row[0], k)
            assert ref["n_nonfinite"] == ref["n_nonphys"] == 0
