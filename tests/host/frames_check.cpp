// Checks the frames and the patches of pdbm_offsets.h on the host, as the
// kernels evaluate them:
//   - octant_by (a multiplication) equals octant_of (integer division) and
//     wrap_col the modulo, over whole small grids and around every octant
//     boundary and end of the largest;
//   - the turns of strip_turns and of a strip's lanes are those of turn_of,
//     the halo gather of the upwind planes reads inside f and the planes the
//     neighbour holds them in;
//   - the patches of a grid own every cell once, load inside the grid, and a
//     cell still needed finds its true neighbours, in their frames.
// Exit status 0 when all hold.
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

static void column(int col, int nt, int s)
{
    const double inv2 = 0.5 / nt;
    check(octant_by(col, inv2, s) == octant_of(col, nt, s), "octant", col, nt, s, 0);
    check(wrap_col(col, nt, inv2) == ((col % nt) + nt) % nt, "wrap", col, nt, s, 0);
}

static void strips(int nt, int s, int esz)
{
    const int64_t pitch = (nt + STRIP - 1) / STRIP * STRIP;
    const RowBytes b = row_bytes_of(NQ * pitch, pitch, esz);
    for (int strip = 0; strip * STRIP < nt; ++strip) {
        const int c0 = strip * STRIP;
        const StripTurns t = strip_turns(0.5 / nt, s, strip);
        for (int side = 0; side < 2; ++side) {
            const int k = side ? c0 + 63 : c0, c = side ? c0 + 64 : c0 - 1;
            check(t.tc[side] == turn_of(k, c, nt, s) && t.tl[side] == turn_of(c, c - 1, nt, s) &&
                      t.tr[side] == turn_of(c, c + 1, nt, s),
                  "edge turn", nt, s, strip, side);
        }
        bool any = false;
        for (int lane = 0; lane < 64; ++lane) {
            const StripOffsets o = strip_offsets(nt, pitch, s, true, esz, b, strip, lane);
            const int col = c0 + lane;
            check(o.turn_left == (lane > 0 && turn_of(col, col - 1, nt, s) != 0), "lane left", nt, s, strip, lane);
            check(o.turn_right == (lane < 63 && turn_of(col, col + 1, nt, s) != 0), "lane right", nt, s, strip, lane);
            // marched grids turn by at most one octant, away from it on the left, into it on the right
            if (o.turn_left) check(turn_of(col, col - 1, nt, s) == 1, "left turn", nt, s, strip, lane);
            if (o.turn_right) check(turn_of(col, col + 1, nt, s) == 7, "right turn", nt, s, strip, lane);
            any = any || o.turn_left || o.turn_right;
            const int left = (lane & 16) == 0, dd = lane & 3, ring = (lane & 15) >> 2;
            const int c = left ? c0 - 1 : c0 + 64, dir = left ? left_dir(dd) : right_dir(dd);
            const int q = plane_of(1 + 8 * ring + dir, turn_of(left ? c0 : c0 + 63, c, nt, s));
            check(o.vhs == elem_of(q, ((c % nt) + nt) % nt, pitch) * esz && o.vhs + esz <= b.row, "upwind gather", nt, s,
                  strip, lane);
        }
        if (whole_octants(nt, s)) check(!any, "whole octants", nt, s, strip, 0);
    }
}

static void patches(int nr, int nt, int s, const PatchGeom &g)
{
    std::vector<int> owned((size_t)nr * nt, 0);
    const int cells = g.threads / g.lanes;
    for (int tile = 0; tile < g.ntiles; ++tile) {
        std::vector<PatchCell> P;
        for (int i = 0; i < cells; ++i) P.push_back(patch_cell(g, nr, nt, 0.5 / nt, tile, i));
        check(P[0].nrow * P[0].ncol <= cells, "patch fits", nr, nt, s, tile);
        for (int i = 0; i < cells; ++i) {
            const PatchCell &c = P[i];
            check(c.row >= 0 && c.row < nr && c.pc >= 0 && c.pc < nt, "loads inside", nr, nt, tile, i);
            check(c.pc == ((c.ext % nt) + nt) % nt, "image", nr, nt, tile, i);
            const PatchNear p = patch_near(c, 0.5 / nt, nt, s, i);
            for (int j : {p.low, p.high, p.left, p.right}) check(j >= 0 && j < cells, "place", nr, nt, tile, i);
            if (c.own) {
                ++owned[(size_t)c.row * nt + c.pc];
                check(c.dist >= g.k, "own cells are a halo in", nr, nt, tile, i);
            }
            if (c.dist < 1) continue;
            // needed at some step: each neighbour is held, one step less far in at most
            check(P[p.low].row == (c.row > 0 ? c.row - 1 : 0) && P[p.low].ext == c.ext, "below", nr, nt, tile, i);
            check(P[p.high].row == (c.row < nr - 1 ? c.row + 1 : nr - 1) && P[p.high].ext == c.ext, "above", nr, nt, tile,
                  i);
            check(P[p.left].row == c.row && P[p.left].pc == (((c.ext - 1) % nt) + nt) % nt, "left", nr, nt, tile, i);
            check(P[p.right].row == c.row && P[p.right].pc == (c.ext + 1 + nt) % nt, "right", nr, nt, tile, i);
            for (int j : {p.low, p.high, p.left, p.right})
                check(P[j].dist >= c.dist - 1, "neighbour still true", nr, nt, tile, i);
            check(p.turn_left == turn_of(c.ext, c.ext - 1, nt, s) && p.turn_right == turn_of(c.ext, c.ext + 1, nt, s),
                  "turn", nr, nt, tile, i);
        }
    }
    for (size_t i = 0; i < owned.size(); ++i) check(owned[i] == 1, "owned once", nr, nt, s, (long)i);
}

int main()
{
    for (int s = 1; s <= 8; ++s) {
        for (int nt = 1; nt <= 700; ++nt)
            for (int c = -70; c < nt + 140; ++c) column(c, nt, s);
        for (int nt : {1 << 24, (1 << 24) - 1, 16777213, 8388608, 4194303, 65536, 4000, 1935})
            for (int k = 0; k <= s; ++k)
                for (int d = -80; d < 140; ++d) {
                    const long c = (long)nt * k / s + d;
                    if (c >= -70 && c < nt + 140) column((int)c, nt, s);
                }
        for (int nt : {8, 9, 15, 16, 17, 63, 64, 65, 100, 127, 128, 129, 200, 256, 512, 513, 1024, 1935})
            for (int esz : {4, 8})
                if (marchable(nt, s)) strips(nt, s, esz);
        for (int nr : {1, 2, 5, 17, 64, 130})
            for (int nt : {1, 2, 3, 4, 5, 7, 8, 17, 33, 64, 65, 130}) {
                for (int form = 0; form < 4; ++form) {
                    const PatchGeom g = patch_geom(nr, nt, s, form & 1, form & 2);
                    if (g.threads) patches(nr, nt, s, g);
                    else check(marchable(nt, s) || nt == 1, "every grid has a kernel", nr, nt, s, form);
                }
                // and patches of other shapes: cut both ways, closing the ring, one cell
                for (int rows : {1, 4, 9})
                    for (int cols : {1, 4, 8, nt})
                        for (int k : {1, 2, 3}) {
                            PatchGeom o{rows, cols < nt ? cols : nt, k, 0, 0, 512, 4};
                            o.nbc = (nt + o.cols - 1) / o.cols;
                            o.ntiles = o.nbc * ((nr + rows - 1) / rows);
                            const int ncol = o.cols >= nt ? nt : o.cols + 2 * k;
                            if ((rows + 2 * k) * ncol * o.lanes <= o.threads) patches(nr, nt, s, o);
                        }
            }
    }
    // every shape of the rule, on grids at the ends of its ranges
    for (bool fp32 : {false, true})
        for (int nr : {1, 9, 64, 100, 300, 700})
            for (int nt : {8, 15, 16, 17, 20, 64, 130, 200, 333}) {
                const PatchGeom g = patch_geom(nr, nt, 8, fp32, true);
                if (g.threads) patches(nr, nt, 8, g);
            }
    for (int nr : {1, 79, 80, 81, 20000, 40960, 40961}) {
        const PatchGeom g = patch_geom(nr, 1, 8, false, true);
        check((g.threads != 0) == (nr <= 40960), "column limit", nr, g.threads, 0, 0);
        if (g.threads) patches(nr, 1, 8, g);
    }
    std::printf("%lld checks, %lld failed\n", n, bad);
    return bad ? 1 : 0;
}
