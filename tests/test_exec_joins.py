"""Build-level check that needs no GPU, on the gfx950 assembly of every kernel:
where the lanes of a divergent branch come together again (a label that a
branch around the region with no lane left jumps to), no vector instruction
runs before the lane mask is restored.  A live value copied there, as the
register allocator has done in a kernel full of live registers, is copied in
the lanes that took the branch only, and the others later read a stale copy."""
import glob
import os
import re
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

from paper_1308_0653_amd import build as B


def _early_vector_ops(lines):
    """(label, instruction) of the vector instructions between a join's label
    and the restore of the lane mask.  Moves of spilled scalar registers
    (v_readlane, v_writelane) do not depend on the mask."""
    targets = {m.group(1) for t in lines if (m := re.match(r"\s*s_cbranch_exec\w+\s+(\.LBB\S+)", t))}
    out, label, seen = [], None, []
    for line in lines:
        m = re.match(r"^(\.LBB\S+):", line)
        if m:
            label, seen = (m.group(1) if m.group(1) in targets else None), []
            continue
        t = line.split(";")[0].strip()
        if label is None or not t:
            continue
        if re.match(r"s_or_b64\s+exec,\s*exec", t):
            out += [(label, v) for v in seen]
            label = None
        elif re.match(r"s_(cbranch\w*|branch|endpgm|\w+_saveexec_b64)\b", t):
            label = None
        elif re.match(r"(v_(?!readlane|writelane)|ds_|buffer_|global_|flat_)", t):
            seen.append(t)
    return out


def test_check_finds_a_copy_before_the_restore():
    copy = "v_accvgpr_write_b32 a20, v120"
    region = ["s_and_saveexec_b64 s[54:55], vcc", "s_cbranch_execz .LBB4_189", "v_mul_f64 v[0:1], v[2:3], v[4:5]",
              ".LBB4_189:", "s_mov_b64 s[72:73], s[92:93]", "s_or_b64 exec, exec, s[54:55]", "v_mov_b32 v0, v1"]
    assert _early_vector_ops(region) == []
    assert _early_vector_ops(region[:4] + [copy] + region[4:]) == [(".LBB4_189", copy)]
    assert _early_vector_ops(region[:4] + ["v_readlane_b32 s18, v253, 0"] + region[4:]) == []


def test_no_vector_instruction_before_the_lane_mask_is_restored():
    def asm(src):
        with tempfile.TemporaryDirectory() as tmp:
            dst = os.path.join(tmp, "k.s")
            cmd = [B.HIPCC, *[f for f in B.FLAGS if f not in ("-shared", "-fPIC")], f"-I{B.INCLUDE}", f"-I{B.CSRC}",
                   "--cuda-device-only", "-S", src, "-o", dst]
            subprocess.run(cmd, cwd=tmp, check=True, capture_output=True)
            return open(dst).read()

    with ThreadPoolExecutor(4) as pool:
        texts = list(pool.map(asm, sorted(glob.glob(os.path.join(B.CSRC, "*.hip")))))
    kernels, found = 0, []
    for text in texts:
        for m in re.finditer(r"^(_ZN4pdbm\S*k_[a-z]\S*):", text, flags=re.M):
            kernels += 1
            body = text[m.end():text.index(".Lfunc_end", m.end())].split("\n")
            found += [(m.group(1), *x) for x in _early_vector_ops(body)]
    assert kernels >= 30 and not found, found
