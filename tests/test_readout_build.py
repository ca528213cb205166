"""Build-level check that needs no GPU, on the gfx950 assembly of the read-out
kernels: the sums of k_noneq over the velocities are fused multiply-adds, one
per velocity and measure, and k_moments forms T and the polar velocities with
them (nothing is fused by the compiler in these sources)."""
import os
import re
import subprocess
import tempfile

from paper_1308_0653_amd import build as B
from tests.test_build import _kernel_bodies


def test_read_outs_sum_with_fused_multiply_adds():
    with tempfile.TemporaryDirectory() as tmp:
        dst = os.path.join(tmp, "cells.s")
        cmd = [B.HIPCC, *[f for f in B.FLAGS if f not in ("-shared", "-fPIC")], f"-I{B.INCLUDE}", f"-I{B.CSRC}",
               "--cuda-device-only", "-S", os.path.join(B.CSRC, "pdbm_cells.hip"), "-o", dst]
        subprocess.run(cmd, cwd=tmp, check=True, capture_output=True)
        asm = open(dst).read()

    def fused(lines, real):
        return sum(bool(re.match(rf"\s*v_fmac?_{real}", t)) for t in lines)

    noneq = list(_kernel_bodies(asm, "k_noneq"))
    assert len(noneq) == 2
    for name, lines in noneq:
        # 12 measures of 32 moving velocities
        assert fused(lines, "f64") >= 12 * 32, (name, fused(lines, "f64"))
    # float32 k_moments: the direction sums of 4 rings (2 each), the sums over
    # the speeds (2 each of 3), and T's two
    (name, lines), = [x for x in _kernel_bodies(asm, "k_moments") if "k_momentsIf" in x[0]]
    divisions = sum("v_div_scale_f32" in t for t in lines) // 2  # 4 of each are theirs at the least
    assert fused(lines, "f32") >= 8 + 6 + 2 + 4 * divisions, (name, fused(lines, "f32"), divisions)
