// Byte offsets of the raw buffer accesses of the step kernels: plain integer
// arithmetic, shared by the kernels (pdbm_device.h, pdbm_step.hip,
// pdbm_step2.hip) and by the host bounds check (tests/host/offsets_check.cpp,
// built with g++ from this header), which evaluates the same functions for
// every lane, strip and row of a grid and checks each access against its
// buffer.
//
// A buffer access reads or writes at base + so + vo, so = a scalar (row)
// offset, vo = a per-lane offset, both 32-bit: each f buffer stays below
// 4 GiB (checked at create).
#pragma once

#include <math.h>
#include <stdint.h>

#include "pdbm_internal.h"

namespace pdbm {

// Frames.  Column j keeps its directions relative to its octant o(j), the
// multiple of pi/4 at or below theta_j: "direction i" of a cell means the
// Cartesian direction (i + o) % 8, at angle i pi/4 - theta' to e_r with
// theta' = theta_j - o pi/4 in [0, pi/4).  In that frame the signs of all
// velocity components are the same in every column: directions 0, 1, 2, 7
// point outward (C_r >= 0, upwind neighbour below), 3 to 6 inward; 1 to 4
// point along +theta (upwind neighbour on the left), 5, 6, 7, 0 along -theta.
// Columns are numbered on past the ends of the sector: column nt is the image
// of column 0 one sector further round, its data that of column 0, its octant
// o(0) + sector.  So the rotated periodic halo of Sec. II.D is the plain rule
// between neighbouring columns, in or out of the grid: direction i of column
// c is direction i + o(c) - o(c') of column c'.
__host__ __device__ constexpr int wraps_of(int c, int n) { return c >= 0 ? c / n : -((n - 1 - c) / n); }  // floor(c / n)
__host__ __device__ constexpr int octant_of(int col, int nt, int sector)
{
    return wraps_of((2 * col + 1) * sector, 2 * nt);
}
// The same without an integer division, with inv2 = 1 / (2 nt): octants are
// multiples of 1 / (2 nt) >= 2^-26 apart, the product is off by under 2^-47.
__host__ __device__ inline int octant_by(int col, double inv2, int sector)
{
    return (int)floor((double)((2 * col + 1) * sector) * inv2 + 0x1p-27);
}
// Shift of direction indices from column `from` to its neighbour `to`.
__host__ __device__ constexpr int turn_of(int from, int to, int nt, int sector)
{
    return (octant_of(from, nt, sector) - octant_of(to, nt, sector)) & 7;
}
// Whether neighbouring columns differ by at most one octant (what the
// marching kernels take; narrower grids are stepped on patches), and whether
// none do so within a strip.
__host__ __device__ constexpr bool marchable(int nt, int sector) { return nt >= sector; }
__host__ __device__ constexpr bool whole_octants(int nt, int sector) { return nt % (STRIP * sector) == 0; }

// Column c (a little off the grid at most) as a column of the grid.
__host__ __device__ inline int wrap_col(int c, int nt, double inv2) { return c - nt * octant_by(c, inv2, 1); }

// Plane of velocity q of a neighbour whose frame is turned by r.
__host__ __device__ constexpr int plane_of(int q, int r)
{
    return q == 0 ? 0 : 1 + 8 * ((q - 1) / 8) + ((((q - 1) % 8) + r) & 7);
}
// The member of pair dd that comes from the left and from the right (see
// above), and the one that comes from below.
__host__ __device__ constexpr int left_dir(int dd) { return dd == 0 ? 4 : dd; }
__host__ __device__ constexpr int right_dir(int dd) { return dd == 0 ? 0 : dd + 4; }
__host__ __device__ constexpr int low_dir(int dd) { return dd == 3 ? 7 : dd; }

// Row strides of one solve, in bytes.
struct RowBytes {
    uint32_t row;   // one r row of f: NQ planes of pitch values
    uint32_t lrow;  // one r row of lambda: pitch doubles
    uint32_t rest;  // the rest particle's plane (pitch values); also one row of the per-cell tau field
    uint32_t pair;  // one pair of opposite directions (2 pitch values)
};
__host__ __device__ inline RowBytes row_bytes_of(int64_t rstride, int64_t pitch, int esz)
{
    RowBytes b;
    b.row = (uint32_t)rstride * (uint32_t)esz;
    b.lrow = (uint32_t)pitch * 8u;
    b.rest = (uint32_t)pitch * (uint32_t)esz;
    b.pair = 2u * b.rest;
    return b;
}

// How frames turn at the two edges of a strip: of the columns bordering it
// on the left [0] and the right [1], the shifts of direction indices from the
// strip's lane beside it to it (tc) and from it to its own neighbours (tl,
// tr).  (Read from a table instead of worked out here, the longer chain of
// loads ahead of a wavefront's gathers cost float32 launches 2 %.)
struct StripTurns {
    int tc[2], tl[2], tr[2];
};
__host__ __device__ inline StripTurns strip_turns(double inv2, int sector, int strip)
{
    StripTurns t;
    for (int side = 0; side < 2; ++side) {
        const int k = side == 0 ? strip * STRIP : strip * STRIP + STRIP - 1, c = side == 0 ? k - 1 : k + 1;
        const int ok = octant_by(k, inv2, sector), oc = octant_by(c, inv2, sector);
        const int far = octant_by(side == 0 ? c - 1 : c + 1, inv2, sector);
        t.tc[side] = (ok - oc) & 7;
        t.tl[side] = (oc - (side == 0 ? far : ok)) & 7;
        t.tr[side] = (oc - (side == 0 ? ok : far)) & 7;
    }
    return t;
}

// Per-lane offsets of a wavefront strip (see Strip in pdbm_device.h): lane
// `lane` of strip `strip` owns column c0 + lane, c0 = 64 strip, or its
// periodic image (the data of physical column pc).  `mixed`: the strip may
// hold columns of more than one octant.
struct StripOffsets {
    uint32_t vo, vo2, vol;     // this lane's physical column: rest plane, pair, lambda
    uint32_t vos, vos2, vols;  // ... of its own column (the padding for periodic images)
    uint32_t vh1, vh2, vhl;    // halo gathers of every plane (plane and column)
    uint32_t vhs;              // halo gather of the upwind planes: lanes 0..15 left, 16..31 right, pair lane % 16
    uint32_t poff[4];          // the lane's pairs of the slowest speed
    int pc;
    bool turn_left, turn_right;  // the lane's neighbour in the strip lies in the octant before or after
    bool useful;               // the lane holds a grid column (not an image)
};
__host__ __device__ inline StripOffsets strip_offsets(const StripTurns &t, double inv2, int nt, int64_t pitch,
                                                      int sector, bool mixed, int esz, const RowBytes &b, int strip,
                                                      int lane)
{
    StripOffsets o;
    const int c0 = strip * STRIP;
    const int col = c0 + lane;
    // lanes past the last column hold periodic images of the first ones
    o.pc = wrap_col(col, nt, inv2);
    o.useful = col < nt;
    o.vo = (uint32_t)o.pc * (uint32_t)esz;
    o.vo2 = 2u * o.vo;
    o.vol = (uint32_t)o.pc * 8u;
    o.vos = (uint32_t)col * (uint32_t)esz;
    o.vos2 = 2u * o.vos;
    o.vols = (uint32_t)col * 8u;
    for (int dd = 0; dd < 4; ++dd) o.poff[dd] = o.vo2 + b.rest + (uint32_t)dd * b.pair;
    const int oct = octant_by(col, inv2, sector);  // (each worked out by every lane, whatever the others say)
    const bool tl = octant_by(col - 1, inv2, sector) != oct, tr = octant_by(col + 1, inv2, sector) != oct;
    o.turn_left = mixed && lane > 0 && tl;
    o.turn_right = mixed && lane < STRIP - 1 && tr;
    // halo columns: c0 - 1 and c0 + 64, as periodic images
    const int cl = wrap_col(c0 - 1, nt, inv2), rl = t.tc[0];
    const int cr = wrap_col(c0 + STRIP, nt, inv2), rr = t.tc[1];
    // gather 1: lanes 0..32 left halo of planes 0..32, lanes 33..63 right
    // halo of planes 0..30; gather 2: lanes 0, 1 right halo of planes 31,
    // 32; lambda gather: lane 0 left, lane 1 right (other lanes repeat a
    // valid address)
    o.vh1 = lane <= 32 ? (uint32_t)elem_of(plane_of(lane, rl), cl, pitch) * (uint32_t)esz
                       : (uint32_t)elem_of(plane_of(lane - 33, rr), cr, pitch) * (uint32_t)esz;
    o.vh2 = lane < 2 ? (uint32_t)elem_of(plane_of(31 + lane, rr), cr, pitch) * (uint32_t)esz
                     : (uint32_t)cl * (uint32_t)esz;
    o.vhl = lane == 1 ? (uint32_t)cr * 8u : (uint32_t)cl * 8u;
    // the upwind halves of them
    const int k = (lane & 15) >> 2, dd = lane & 3;
    const bool left = (lane & 16) == 0;
    const int q = plane_of(1 + 8 * k + (left ? left_dir(dd) : right_dir(dd)), left ? rl : rr);
    o.vhs = (uint32_t)elem_of(q, left ? cl : cr, pitch) * (uint32_t)esz;
    return o;
}
inline StripOffsets strip_offsets(int nt, int64_t pitch, int sector, bool mixed, int esz, const RowBytes &b, int strip,
                                  int lane)
{
    const double inv2 = 0.5 / nt;
    return strip_offsets(strip_turns(inv2, sector, strip), inv2, nt, pitch, sector, mixed, esz, b, strip, lane);
}

// Cells of the two-step kernel's strip edges (edge_cells in pdbm_step2.hip):
// one lane group takes row r of the column bordering strip `strip` on `side`
// (0: left, 1: right) and gathers the cell (row r, column pc), its radial
// neighbours (rows rlo, rhi: zero-gradient ghosts at the ends) and its
// azimuthal neighbours (columns pl, pr), which may be periodic images.
// Direction i of the cell is direction i + tl of its left neighbour, i + tr
// of its right one; direction i of the strip's column beside it (pk) is
// direction i + tc of the cell.
struct EdgeOffsets {
    int pc, pl, pr, pk;            // the cell's column, its left and right neighbours, the column of lane 0 / 63
    int tc, tl, tr, tk;            // shifts of direction indices (tk = 0: the strip's own)
    int rlo, rhi;                  // rows of its radial neighbours
    uint32_t orow, olo, ohi;       // row offsets of f: the cell's row and its radial neighbours
    uint32_t cc, cl, cr;           // pair-column offsets of f: pc, pl, pr
    uint32_t x0;                   // the rest particle of the cell
    uint32_t lc, lb, la, lL, lR;   // lambda: the cell, below, above, left, right
    uint32_t om;                   // the cell's entry of the per-cell tau field
};
__host__ __device__ inline EdgeOffsets edge_offsets(const StripTurns &t, double inv2, int nr, int nt, int esz,
                                                    const RowBytes &b, int strip, int side, int r)
{
    EdgeOffsets o;
    const int c0 = strip * STRIP;
    const int c = side == 0 ? c0 - 1 : c0 + STRIP, k = side == 0 ? c0 : c0 + STRIP - 1;  // strip numbering
    o.pc = wrap_col(c, nt, inv2);
    o.pl = wrap_col(c - 1, nt, inv2);
    o.pr = wrap_col(c + 1, nt, inv2);
    o.pk = wrap_col(k, nt, inv2);
    o.tc = side == 0 ? t.tc[0] : t.tc[1];
    o.tl = side == 0 ? t.tl[0] : t.tl[1];
    o.tr = side == 0 ? t.tr[0] : t.tr[1];
    o.tk = 0;
    o.rlo = r - 1 < 0 ? 0 : r - 1;
    o.rhi = r + 1 > nr - 1 ? nr - 1 : r + 1;
    const uint32_t es = (uint32_t)esz;
    o.orow = (uint32_t)r * b.row;
    o.olo = (uint32_t)o.rlo * b.row;
    o.ohi = (uint32_t)o.rhi * b.row;
    o.cc = 2u * (uint32_t)o.pc * es;
    o.cl = 2u * (uint32_t)o.pl * es;
    o.cr = 2u * (uint32_t)o.pr * es;
    o.x0 = o.orow + (uint32_t)o.pc * es;
    o.lc = (uint32_t)r * b.lrow + (uint32_t)o.pc * 8u;
    o.lb = (uint32_t)o.rlo * b.lrow + (uint32_t)o.pc * 8u;
    o.la = (uint32_t)o.rhi * b.lrow + (uint32_t)o.pc * 8u;
    o.lL = (uint32_t)r * b.lrow + (uint32_t)o.pl * 8u;
    o.lR = (uint32_t)r * b.lrow + (uint32_t)o.pr * 8u;
    o.om = (uint32_t)o.pc * es + (uint32_t)r * b.rest;
    return o;
}
inline EdgeOffsets edge_offsets(int nr, int nt, int sector, bool /*mixed*/, int esz, const RowBytes &b, int strip,
                                int side, int r)
{
    return edge_offsets(strip_turns(0.5 / nt, sector, strip), 0.5 / nt, nr, nt, esz, b, strip, side, r);
}
// Offset of pair i (0..15) within a row of f (column 0).
__host__ __device__ inline uint32_t pair_in_row(const RowBytes &b, int i) { return b.rest + (uint32_t)i * b.pair; }

// The one-step single-column kernel (radial_block in pdbm_step.hip): lane l
// of block blk holds row re = min(COL_W blk + l, nr - 1) of column 0 (it
// owns the rows of lanes below COL_W) and gathers the row below the block
// (rlo, directions turned by `tlo` at the disc centre) and the row 64 above
// its first (rhi).
struct RadialOffsets {
    int re, rlo, rhi;
    uint32_t vo, vol;     // the lane's row: f and lambda
    uint32_t vh1, vh2, vhl;  // gathers of the rows bounding the block
    uint32_t om;             // the lane's entry of the per-cell tau field
};
__host__ __device__ inline RadialOffsets radial_offsets(int nr, int64_t pitch, bool disc, int esz, const RowBytes &b,
                                                        int blk, int lane)
{
    RadialOffsets o;
    const int r0 = blk * COL_W;
    const int row = r0 + lane;
    o.re = row < nr - 1 ? row : nr - 1;  // lanes past the last row hold its zero-gradient image
    o.rlo = r0 == 0 ? 0 : r0 - 1;
    o.rhi = r0 + 64 < nr - 1 ? r0 + 64 : nr - 1;
    const int tlo = r0 == 0 && disc ? 4 : 0;
    const uint32_t es = (uint32_t)esz;
    o.vo = (uint32_t)o.re * b.row;
    o.vol = (uint32_t)o.re * b.lrow;
    o.vh1 = lane <= 32 ? (uint32_t)o.rlo * b.row + (uint32_t)elem_of(plane_of(lane, tlo), 0, pitch) * es
                       : (uint32_t)o.rhi * b.row + (uint32_t)elem_of(lane - 33, 0, pitch) * es;
    o.vh2 = lane < 2 ? (uint32_t)o.rhi * b.row + (uint32_t)elem_of(31 + lane, 0, pitch) * es
                     : (uint32_t)o.rlo * b.row;
    o.vhl = lane == 1 ? (uint32_t)o.rhi * b.lrow : (uint32_t)o.rlo * b.lrow;
    o.om = (uint32_t)o.re * b.rest;
    return o;
}

// The multi-step single-column kernel (k_column in pdbm_step.hip): lane l
// of wavefront t holds row r0 - COL_K + l, r0 = COL_W t, whose data it
// loads from row re (the row clamped to the grid: rows outside it start as
// their radial ghosts), and owns it if it is one of rows r0 .. r0 + COL_W - 1
// of the grid (then it stores the new state there).
struct ColumnOffsets {
    int row, re;
    bool own;
    uint32_t vo, vol, om;  // f (rest plane of the row; pairs follow), lambda, the per-cell tau field
};
__host__ __device__ inline ColumnOffsets column_offsets(int nr, const RowBytes &b, int t, int lane)
{
    ColumnOffsets o;
    const int r0 = t * COL_W;
    o.row = r0 - COL_K + lane;
    o.re = o.row < 0 ? 0 : o.row > nr - 1 ? nr - 1 : o.row;
    o.own = lane >= COL_K && lane < COL_K + COL_W && o.row < nr;
    o.vo = (uint32_t)o.re * b.row;
    o.vol = (uint32_t)o.re * b.lrow;
    o.om = (uint32_t)o.re * b.rest;
    return o;
}

// The patches of the multi-step kernel for small grids (k_patch in
// pdbm_patch.hip): workgroup `tile` of a solve owns rows x cols cells of the
// grid and holds them with a halo of k rows and columns, `lanes` lanes to a
// cell, cells row by row.  Rows are clipped to the grid; with cols >= nt
// the patch holds the whole ring and has no column halo.
// Shapes of patches a solve alone on the GPU chooses from (patch_geom):
// the cells of a workgroup (rows x cols, halo included), its threads, lanes
// per cell and halo k, and what a launch takes in ns, t0 + rounds c with 256
// workgroups to a round, one per CU, fitted to grids of 100 x 100 to 400 x
// 300 cells.
struct PatchShape {
    int rows, cols, k, threads, lanes, t0, c;
};
constexpr PatchShape PATCH_FP64[] = {
    {16, 16, 2, 512, 2, 2500, 6400}, {16, 16, 3, 512, 2, 2800, 8400}, {16, 16, 4, 512, 2, 3200, 9200},
    {10, 10, 3, 512, 4, 2800, 5000}};
constexpr PatchShape PATCH_FP32[] = {
    {16, 16, 2, 512, 2, 2700, 5000}, {16, 16, 3, 512, 2, 3000, 6100},  {16, 16, 4, 512, 2, 3000, 6800},
    {12, 12, 4, 768, 4, 2800, 6000}, {19, 20, 3, 768, 2, 3000, 10500}};
// Grids of fewer columns than octants, alone or packed: NARROW, and with
// drift records NARROW_TALL instead of more than NARROW_MOST patches.  A
// patch keeps a drift partial sum per step; a tall one owns 32 rows or more,
// so that these sums take no more memory than those of wavefronts marching 16
// rows.  Per step, tall against not: 64 x 4 4.2 against 3.2 us (float64) and
// 3.6 / 3.1 (float32), 4000 x 5 4.9 / 4.3 and 4.2 / 3.9, 20000 x 6 17.6 / 17.1
// and 14.4 / 13.4, 40000 x 7 29.9 / 38.2 and 23.7 / 27.2.
constexpr PatchShape NARROW = {8, 8, 2, 256, 4, 0, 0}, NARROW_TALL = {32, 8, 2, 512, 2, 0, 0};
constexpr int NARROW_MOST = 1024;
// One theta column: 128 rows, 24 steps.
constexpr PatchShape PATCH_COLUMN = {128, 1, 24, 256, 2, 0, 0};
// Rounds up to which patches are the faster: of the 16 x 16 shape with k = 2
// (110 thousand cells), and of the column's (41 thousand rows).
constexpr int PATCH_ROUNDS = 3, PATCH_COLUMN_ROUNDS = 2;

inline PatchGeom patches_of(const PatchShape &s, int nr, int nt)
{
    PatchGeom g{};
    g.k = s.k;
    g.threads = s.threads;
    g.lanes = s.lanes;
    if (nt <= s.cols) {  // the patch closes the ring and takes more rows instead
        g.cols = nt;
        g.rows = s.rows * s.cols / nt - 2 * s.k;
    } else {
        g.cols = s.cols - 2 * s.k;
        g.rows = s.rows - 2 * s.k;
    }
    g.nbc = (nt + g.cols - 1) / g.cols;
    g.ntiles = g.nbc * ((nr + g.rows - 1) / g.rows);
    return g;
}
// Patches of a grid (`alone` on the GPU, or in a pack; with drift `records`
// or not); threads = 0: it has none and is marched by wavefronts or, a single column, held by them.
// - Fewer columns than octants: always, as neighbouring columns may then
//   differ by more than the one octant the marching kernels take.
// - Alone and too small to fill the GPU with marching wavefronts: a launch of
//   those takes as long as one wavefront's chain of rows however few there
//   are, 25 us in float64 and 20 us in float32 for two steps of up to 60
//   thousand cells.  Patches took, per step, against marching: 64 x 64 2.6
//   against 12.2 us (float64), 2.2 against 9.8 (float32); 100 x 100 3.2 / 12.6
//   and 2.4 / 10.1; 300 x 130 6.4 / 13.2 and 4.5 / 10.4; 300 x 200 8.1 / 13.8
//   and 6.3 / 10.4; 400 x 300 16.1 / 15.3 and 11.6 / 10.9 (marched).  A single
//   column of 20000 rows: 2.0 against 3.6 us (float64), 1.6 against 2.6.
inline PatchGeom patch_geom(int nr, int nt, int sector, bool fp32, bool alone, bool records = false)
{
    if (nt > 1 && !marchable(nt, sector)) {
        const PatchGeom g = patches_of(NARROW, nr, nt);
        return records && g.ntiles > NARROW_MOST ? patches_of(NARROW_TALL, nr, nt) : g;
    }
    if (!alone) return PatchGeom{};
    if (nt == 1) {
        const PatchGeom g = patches_of(PATCH_COLUMN, nr, 1);
        return g.ntiles <= 256 * PATCH_COLUMN_ROUNDS ? g : PatchGeom{};
    }
    const PatchShape *shapes = fp32 ? PATCH_FP32 : PATCH_FP64;
    const int n = fp32 ? (int)(sizeof PATCH_FP32 / sizeof *PATCH_FP32) : (int)(sizeof PATCH_FP64 / sizeof *PATCH_FP64);
    if (patches_of(shapes[0], nr, nt).ntiles > 256 * PATCH_ROUNDS) return PatchGeom{};
    PatchGeom best{};
    double least = 0.0;
    for (int i = 0; i < n; ++i) {
        const PatchGeom g = patches_of(shapes[i], nr, nt);
        const double ns = (shapes[i].t0 + (double)((g.ntiles + 255) / 256) * shapes[i].c) / shapes[i].k;
        if (i == 0 || ns < least) {
            best = g;
            least = ns;
        }
    }
    return best;
}
// Whether single steps of a grid on patches `g`, alone on the GPU, are marched
// all the same (rows_one): the 16 x 16 shape with k = 2 takes more than two
// rounds, and the patches' kernel clears what a record of the two forms leaves
// unused (those of four lanes to a cell, for smaller grids, need not).
__host__ __device__ constexpr bool marched_beside(int lanes) { return lanes == 2; }
inline bool single_steps_march(int nr, int nt, int sector, bool fp32, const PatchGeom &g)
{
    return nt > 1 && marchable(nt, sector) && marched_beside(g.lanes) &&
           patches_of(fp32 ? PATCH_FP32[0] : PATCH_FP64[0], nr, nt).ntiles > 256 * 2;
}
struct PatchCell {
    int row, pc, ext;    // its row, physical column, column before wrapping
    int lr, lc, nrow, ncol;  // place within the patch, rows and columns of the patch
    int dist;            // how far in from the edge of the halo it sits (-1: no cell, the lane is idle)
    bool own;            // the patch stores it
    bool ring;           // the patch holds the whole ring
};
__host__ __device__ inline PatchCell patch_cell(const PatchGeom &g, int nr, int nt, double inv2, int tile,
                                                int cell)
{
    PatchCell c;
    const int rb = tile / g.nbc, cb = tile - rb * g.nbc;
    const int r0 = rb * g.rows, r1 = r0 + g.rows < nr ? r0 + g.rows : nr;
    const int rlo = r0 - g.k > 0 ? r0 - g.k : 0, rhi = r1 + g.k < nr ? r1 + g.k : nr;
    c.ring = g.cols >= nt;
    const int c0 = cb * g.cols, c1 = c0 + g.cols < nt ? c0 + g.cols : nt;
    const int clo = c.ring ? 0 : c0 - g.k;
    c.nrow = rhi - rlo;
    c.ncol = c.ring ? nt : c1 - c0 + 2 * g.k;
    c.lr = cell / c.ncol;
    c.lc = cell - c.lr * c.ncol;
    const bool in = c.lr < c.nrow;
    if (!in) c.lr = c.lc = 0;
    c.row = rlo + c.lr;
    const int ext = c.ext = clo + c.lc;
    c.pc = wrap_col(ext, nt, inv2);
    const int far = 1 << 20;
    const int below = rlo > 0 ? c.lr : far, above = rhi < nr ? c.nrow - 1 - c.lr : far;
    const int left = c.ring ? far : c.lc, right = c.ring ? far : c.ncol - 1 - c.lc;
    const int dr = below < above ? below : above, dc = left < right ? left : right;
    c.dist = !in ? -1 : dr < dc ? dr : dc;
    c.own = in && c.row >= r0 && c.row < r1 && ext >= c0 && ext < c1;
    return c;
}
// Byte offsets of what lane h of a cell's `lanes` loads and stores: the first of
// its 16 / lanes pairs (each next one a pair on), the rest particle, lambda and
// the cell's entry of the per-cell tau field.
struct PatchOffsets {
    uint32_t pair, rest, lam, om;
};
__host__ __device__ inline PatchOffsets patch_offsets(const PatchCell &c, const RowBytes &b, int esz, int lanes, int h)
{
    PatchOffsets o;
    const uint32_t es = (uint32_t)esz, row = (uint32_t)c.row * b.row;
    o.rest = row + (uint32_t)c.pc * es;
    o.lam = (uint32_t)c.row * b.lrow + (uint32_t)c.pc * 8u;
    o.pair = row + 2u * (uint32_t)c.pc * es + pair_in_row(b, 16 / lanes * h);
    o.om = (uint32_t)c.row * b.rest + (uint32_t)c.pc * es;
    return o;
}
// Places (cells of the patch) of a cell's neighbours: itself beyond the
// radial ends of the grid (the ghosts of Sec. II.D) and at the edge of the
// halo (never used by a cell still needed), the other end around a whole
// ring; and the shifts of direction indices to the azimuthal ones.
struct PatchNear {
    int low, high, left, right, turn_left, turn_right;
};
__host__ __device__ inline PatchNear patch_near(const PatchCell &c, double inv2, int nt, int sector, int cell)
{
    PatchNear p;
    const bool in = c.dist >= 0;
    p.low = in && c.lr > 0 ? cell - c.ncol : cell;
    p.high = in && c.lr < c.nrow - 1 ? cell + c.ncol : cell;
    p.left = in && c.lc > 0 ? cell - 1 : in && c.ring ? cell + nt - 1 : cell;
    p.right = in && c.lc < c.ncol - 1 ? cell + 1 : in && c.ring ? cell - (nt - 1) : cell;
    const int o = octant_by(c.ext, inv2, sector);
    p.turn_left = (o - octant_by(c.ext - 1, inv2, sector)) & 7;
    p.turn_right = (o - octant_by(c.ext + 1, inv2, sector)) & 7;
    return p;
}

}  // namespace pdbm
