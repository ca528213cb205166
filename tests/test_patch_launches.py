"""How captured steps on patches are cut into launches (patch_launches of
pdbm_schedule.h): every launch takes 1 to `most` steps, they add up, and their
number is even where that of marching launches is."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include "pdbm_schedule.h"
int main()
{
    long bad = 0;
    for (int march : {2, 8})
        for (int most : {1, 2, 3, 4, 24})
            for (int64_t n : {1L, 2L, 3L, 4L, 5L, 6L, 7L, 8L, 9L, 11L, 16L, 23L, 24L, 25L, 47L, 48L, 49L, 200L, 500L, 997L,
                              1L << 40, INT64_MAX}) {
                const int64_t L = pdbm::patch_launches(n, most, march);
                const int64_t m = most > 1 ? n / march + (n % march != 0) : n;
                bad += L < 1 || ((L ^ m) & 1) || L > n || L - 2 > (n - 1) / most;
                if (n > 1000) continue;
                int64_t left = n;
                for (int64_t k = L; k > 0; --k) {
                    const int64_t nk = (left + k - 1) / k;
                    bad += nk < 1 || nk > most;
                    left -= nk;
                }
                bad += left != 0;
            }
    std::printf("%ld bad\n", bad);
    return bad != 0;
}
"""


def test_steps_on_patches_are_cut_into_launches(tmp_path):
    src, exe = tmp_path / "check.cpp", str(tmp_path / "check")
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I" + os.path.join(ROOT, "paper_1308_0653_amd", "csrc"),
                    str(src), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
