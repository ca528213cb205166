// Host bounds check of the patch kernel's accesses and of those of marched
// strips that offsets_check.cpp leaves out, from the functions the kernels use
// (pdbm_offsets.h):
//   - k_patch: every load and store of every lane of every patch (pairs, rest
//     particle, lambda, per-cell tau field), every LDS element of a neighbour,
//     and each value of the grid's columns stored exactly once;
//   - strips of grids with mixed octants: the pairs of load_row and the gather
//     of the upwind halo, in every row.
// The largest grids that take patches of each kind are among them.  Exit
// status 0 when all are inside their buffers.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "pdbm_offsets.h"

using namespace pdbm;

static long long n = 0, bad = 0;
static void check(bool ok, const char *what, long a, long b, long c, long d)
{
    ++n;
    if (!ok && bad++ < 20) std::fprintf(stderr, "FAIL %s: %ld %ld %ld %ld\n", what, a, b, c, d);
}

static int64_t pitch_of(int nt) { return nt == 1 ? 2 : (nt + STRIP - 1) / STRIP * STRIP; }

// A pair access of k_patch: the scalar offset i * b.pair on the lane's.
static void patches(int nr, int nt, int s, int esz, const PatchGeom &g)
{
    const int64_t pitch = pitch_of(nt);
    const RowBytes b = row_bytes_of(NQ * pitch, pitch, esz);
    const uint64_t F = (uint64_t)NQ * nr * pitch * esz, L = (uint64_t)nr * pitch * 8, OM = (uint64_t)nr * pitch * esz;
    check(F < uint64_t(1) << 32, "an accepted grid", nr, nt, esz, 0);
    const int NT = g.threads, LPC = g.lanes, NS = 4 / LPC;
    const bool map = F <= 1 << 24;  // of the values stored
    std::vector<unsigned char> stored(map ? F / esz : 0, 0);
    for (int tile = 0; tile < g.ntiles; ++tile) {
        if (!map && tile > 1000 && tile < g.ntiles - 1000) continue;  // rows in between follow the same steps
        for (int t = 0; t < NT; ++t) {
            const int h = t & (LPC - 1);
            const PatchCell c = patch_cell(g, nr, nt, 0.5 / nt, tile, t / LPC);
            const PatchOffsets o = patch_offsets(c, b, esz, LPC, h);
            for (int i = 0; i < 4 * NS; ++i) {
                const uint64_t at = (uint64_t)o.pair + (uint64_t)i * b.pair;
                check(at + 2 * esz <= F && at % (2 * esz) == 0, "pair", nr, nt, tile, t);
                check(at == (uint64_t)c.row * NQ * pitch * esz + elem_of(1 + 8 * (NS * h + (i >> 2)) + (i & 3), c.pc, pitch) * esz,
                      "pair of its ring", nr, nt, tile, t);
                if (c.own && map) ++stored[at / esz], ++stored[at / esz + 1];
            }
            check((uint64_t)o.rest + esz <= F && o.rest == (uint64_t)c.row * NQ * pitch * esz + (uint64_t)c.pc * esz, "rest",
                  nr, nt, tile, t);
            if (c.own && h == 0 && map) ++stored[o.rest / esz];
            check((uint64_t)o.lam + 8 <= L && o.lam == ((uint64_t)c.row * pitch + c.pc) * 8, "lambda", nr, nt, tile, t);
            check((uint64_t)o.om + esz <= OM && o.om == ((uint64_t)c.row * pitch + c.pc) * esz, "tau field", nr, nt, tile, t);
            // elements of the neighbours' planes, of 8 NS NT, as the kernel forms them (low and low7 at a disc centre)
            const PatchNear p = patch_near(c, 0.5 / nt, nt, s, t / LPC);
            const int turned = c.row == 0 ? 4 * NT : 0;
            for (int kk = 0; kk < NS; ++kk)
                for (int dd = 0; dd < 4; ++dd) {
                    const int ring = kk * 8 * NT;
                    for (int low : {p.low * LPC + h, p.low * LPC + h + turned})
                        if (dd < 3) check(dd * NT + low >= 0 && dd * NT + low < 8 * NT, "below", nr, nt, tile, t);
                    for (int low7 : {p.low * LPC + h, p.low * LPC + h - turned})
                        if (dd == 3) check(7 * NT + low7 >= 0 && 7 * NT + low7 < 8 * NT, "below 7", nr, nt, tile, t);
                    const int high = (dd < 3 ? dd + 4 : dd) * NT + p.high * LPC + h;
                    const int left = ((left_dir(dd) + p.turn_left) & 7) * NT + p.left * LPC + h;
                    const int right = ((right_dir(dd) + p.turn_right) & 7) * NT + p.right * LPC + h;
                    for (int e : {high, left, right})
                        check(e >= 0 && ring + e < 8 * NS * NT, "neighbour", nr, nt, tile, t);
                }
        }
    }
    if (!map) return;
    for (int r = 0; r < nr; ++r)
        for (int q = 0; q < NQ; ++q)
            for (int64_t col = 0; col < pitch; ++col)
                check(stored[r * NQ * pitch + elem_of(q, col, pitch)] == (col < nt), "stored once", nr, nt, r, q);
}

static void strips(int nr, int nt, int s, int esz)
{
    const int64_t pitch = pitch_of(nt);
    const RowBytes b = row_bytes_of(NQ * pitch, pitch, esz);
    const uint64_t F = (uint64_t)NQ * nr * pitch * esz;
    check(F < uint64_t(1) << 32, "an accepted grid", nr, nt, esz, 0);
    for (int strip = 0; strip * STRIP < nt; ++strip)
        for (int lane = 0; lane < 64; ++lane) {
            const StripOffsets o = strip_offsets(nt, pitch, s, !whole_octants(nt, s), esz, b, strip, lane);
            for (int row : {0, 1, nr / 2, nr - 2, nr - 1}) {
                if (row < 0 || row >= nr) continue;
                const uint64_t so = (uint64_t)row * b.row;
                check(so + o.vhs + esz <= F, "upwind halo", nr, nt, row, lane);
                for (int c = 0; c < 16; ++c)
                    check(so + b.rest + (uint64_t)c * b.pair + o.vo2 + 2 * esz <= F, "pair of a row", nr, nt, row, lane);
            }
        }
}

int main()
{
    // grids of fewer columns than octants: patches of both kinds, to the largest
    for (int esz : {4, 8})
        for (int nt = 2; nt <= 7; ++nt) {
            const int most = (int)(((uint64_t(1) << 32) - 1) / ((uint64_t)NQ * pitch_of(nt) * esz));
            for (bool records : {false, true})
                for (int nr : {1, 2, 15, 16, 17, 64, 1023, 5120, 5121, 30000, most}) {
                    const PatchGeom g = patch_geom(nr, nt, 8, esz == 4, false, records);
                    check(g.threads > 0, "patches", nr, nt, records, 0);
                    check(!records || g.ntiles <= NARROW_MOST || g.ntiles <= (nr + FUSE_ROWS - 1) / FUSE_ROWS,
                          "no more records than wavefronts keep", nr, nt, g.ntiles, 0);
                    patches(nr, nt, 8, esz, g);
                }
            patches(200, nt, nt < 4 ? 4 : 8, esz, patch_geom(200, nt, nt < 4 ? 4 : 8, esz == 4, true));
        }
    // grids alone on the GPU: each shape, cut both ways and closing the ring, and the largest
    for (int esz : {4, 8})
        for (int s : {8, 3})
            for (const auto &d : {std::pair<int, int>{1, 9216}, {9216, 12}, {768 * 12, 9}, {64, 64}, {100, 100}, {300, 130},
                                  {200, 180}, {45, 20}, {45, 19}, {130, 16}, {5, 333}, {330, 333}}) {
                const PatchGeom g = patch_geom(d.first, d.second, s, esz == 4, true);
                if (g.threads) patches(d.first, d.second, s, esz, g);
                for (const PatchShape &shape : PATCH_FP64)
                    if (esz == 8) patches(d.first, d.second, s, esz, patches_of(shape, d.first, d.second));
                for (const PatchShape &shape : PATCH_FP32)
                    if (esz == 4) patches(d.first, d.second, s, esz, patches_of(shape, d.first, d.second));
            }
    for (int esz : {4, 8})
        for (int nr : {1, 80, 81, 20000, 40960}) patches(nr, 1, 8, esz, patch_geom(nr, 1, 8, esz == 4, true));
    // strips
    strips(4034, 4000, 8, 8);
    strips(4034, 4000, 7, 8);
    strips(4096, 4096, 3, 4);
    strips(8000, 2000, 5, 4);
    for (int esz : {4, 8})
        for (int nt : {8, 17, 63, 64, 65, 129, 200, 512})
            for (int s : {1, 2, 3, 5, 8})
                for (int nr : {1, 2, 33}) strips(nr, nt, s, esz);
    std::printf("%lld checks, %lld failed\n", n, bad);
    return bad ? 1 : 0;
}
