"""Build-level checks of the patch kernel that need no GPU, as those of the
step kernels: every variant that a shape of patch can select is compiled and
no other, none uses scratch memory, and no DPP move of it runs with lanes
switched off."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_1308_0653_amd import build as B
from tests.test_build import _dpp_under_narrowed_exec, _kernel_bodies

# precision, lanes per cell, threads (PATCH_FP64, PATCH_FP32, PATCH_COLUMN, NARROW and NARROW_TALL of pdbm_offsets.h)
VARIANTS = {(p, lanes, threads) for p in "df" for lanes, threads in [(2, 256), (4, 256), (2, 512)]} | {
    ("d", 4, 512), ("f", 4, 768), ("f", 2, 768)}


@pytest.fixture(scope="module")
def asm():
    with tempfile.TemporaryDirectory() as tmp:
        dst = os.path.join(tmp, "patch.s")
        cmd = [B.HIPCC, *[f for f in B.FLAGS if f not in ("-shared", "-fPIC")], f"-I{B.INCLUDE}", f"-I{B.CSRC}",
               "--cuda-device-only", "-S", os.path.join(B.CSRC, "pdbm_patch.hip"), "-o", dst]
        subprocess.run(cmd, cwd=tmp, check=True, capture_output=True)
        return open(dst).read()


def _variant(name):
    m = re.search(r"k_patchI([df])Lb([01])ELi(\d)ELi(\d+)E", name)
    return m.group(1), int(m.group(3)), int(m.group(4)), m.group(2)


SHAPES = r"""
#include <cstdio>
#include "pdbm_offsets.h"
using namespace pdbm;
static void row(char p, const PatchShape &s) { std::printf("%c %d %d\n", p, s.lanes, s.threads); }
int main()
{
    for (const PatchShape &s : PATCH_FP64) row('d', s);
    for (const PatchShape &s : PATCH_FP32) row('f', s);
    for (const PatchShape &s : {PATCH_COLUMN, NARROW, NARROW_TALL}) row('d', s), row('f', s);
}
"""


def test_shapes_select_compiled_variants(tmp_path):
    src, exe = tmp_path / "shapes.cpp", str(tmp_path / "shapes")
    src.write_text(SHAPES)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + B.INCLUDE,
                    "-I" + B.CSRC, str(src), "-o", exe], check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")
    assert {(p, int(lanes), int(threads)) for p, lanes, threads in (t.split() for t in out if t)} == VARIANTS


def test_no_variant_uses_scratch_memory(asm):
    seen = set()
    for block in asm.split("- .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        seen.add(_variant(name))
        assert int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1)) == 0, name
    assert seen == {(*v, tau) for v in VARIANTS for tau in "01"}


def test_dpp_moves_run_with_every_lane_active(asm):
    bodies = list(_kernel_bodies(asm, "k_patch"))
    assert len(bodies) == 2 * len(VARIANTS)
    for name, lines in bodies:
        # the moments, 4 sums of two words or one from the other lanes of a cell, and the records' 5 sums
        assert sum(bool(re.search(r"\b(row_|quad_perm)", t)) for t in lines) >= 4 + 5 * 6, name
        assert _dpp_under_narrowed_exec(lines) == 0, name
