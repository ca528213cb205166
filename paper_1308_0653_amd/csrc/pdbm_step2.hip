// Two time steps per launch, in one pass over f (k_step2): solves of at least
// a column per octant, any sector (annuli and discs), single or packed, in
// float64 (one wavefront per SIMD) and float32 (two).
#include "pdbm_device.h"

namespace pdbm {
namespace {

// ------------------------------------------------------ two steps per pass --
// Steps s and s + 1 in one pass over f.  Stage A computes the state after
// step s (g) one row ahead of stage B, which computes the state after step
// s + 1 from g and stores it: g never leaves the workgroup.  Stage B's
// azimuthal neighbours of lanes 0 and 63 are g at the columns bordering the
// strip.  Where the strip beside is marched by another wavefront of the
// workgroup (consecutive tiles are strips side by side), that wavefront hands
// them on through LDS, row by row, as its stage A makes them (Beside);
// at the workgroup's ends the wavefront computes those cells itself at the
// start (edge_cells).  With every wavefront computing its own, their gathers
// touched half of f's cache lines a second time in float32 (a quarter in
// float64), and 1024 x 1024 launches took 90 us (135 in float64); now 80 and
// 130, as with no edge cells at all but for 2 us.  A barrier per row in place
// of the counts took 145 us in float64, where a SIMD has no other wavefront
// to run.  A block of R rows runs stage A on R + 2 rows and reads R + 4 rows
// of f; each value is written once per two steps.

// Azimuthal neighbours of lanes 0 and 63 in LDS, read back by every lane: of
// each opposite pair of directions the member that comes from the left
// (lane 0: l[pair], left_dir) and the one that comes from the right (lane 63:
// r[pair], right_dir), and lambda.  For stage A the gathered halo of its row
// (slots 0..15 and 16..31 of the wavefront's halo row), for stage B the edge
// cells of the intermediate state.
template <typename real>
struct Halo {
    const real *l, *r;
    double ll, lr;
};
// The gathered halo registers of one row (see Strip::load_upwind_halo).
template <typename real>
struct GatherHalo {
    real h;
    double hl;
};

// Drift sums of one step (mass, energy, chemical energy, non-finite and
// non-physical cells; see diag_cell), kept per lane over the whole march and
// added across the wavefront at the end.  In float32 they take 20 of the
// kernel's 256 registers; summing each row across the wavefront at once
// instead (a DPP reduction per row, no registers held) took 1.9 % more time.
struct LaneDiag {
    double red[5] = {0, 0, 0, 0, 0};
    __device__ __forceinline__ void add(bool valid, double rho, double ux, double uy, double T, double e, double lam,
                                        double w, double Q)
    {
        diag_cell(red, valid, rho, ux, uy, T, e, lam, w, Q);
    }
    __device__ __forceinline__ double total(int i) const { return wave_sum(red[i]); }
};

// One row of one of the two steps, marching outward: the arithmetic of
// update_row with every upwind side known at compile time (the frames of
// pdbm_offsets.h): below for directions 0, 1, 2, 7, above for 3 to 6, left
// for 1 to 4, right for 5, 6, 7, 0.  That is one lane shift per direction and
// no selects, half the LDS reads of the row ahead and of the halo, and no
// lane masks to hold (with both sides fetched and selected per lane, 1024 x
// 1024 launches took 155 us in float64 and 94 us in float32, then 140 and
// 91).  MIXED strips, where a lane's neighbour may lie in the octant
// beside, shift one value more per side and ring and select between the two.
// Radial neighbours: the row behind (below) in compact LDS slots (low_dir of
// each pair, slot 4 (k - 1) + (direction mod 4); replaced by this row's as
// they are read), the row ahead in `fn` (stage A) or in the full LDS row `ga`
// (stage B).  STAGEA: the new row goes to `ga` and `lout`, for every lane
// (stage B reads the periodic images too), and the row it replaces in `ga` to
// `gold`, plane by plane, so that the registers of the old row fill as those
// of fc empty; otherwise it is stored, for the strip's own columns.
template <typename real, bool STAGEA, bool TAUF, bool MIXED, class Diag>
__device__ __forceinline__ void stage_row(const Strip<real, MIXED> &S, int ir, real (*behind)[64], const real fc[NQ],
                                          const real *fn, real (*ga)[64], real *gold, const Halo<real> &H,
                                          double lbehind, double lc, double lahead, const real acr[4],
                                          const real ctv[4], double2 cs, double &lout, real om, Diag &D, bool diag)
{
    const DescPtr dp = S.dp;
    // the cell's exp(-dt/tau): with TAUF `om`, loaded by march2 a pass ahead
    real omega;
    if constexpr (TAUF)
        omega = om;
    else
        omega = omega_at<real, TAUF>(dp, S.vo, (uint32_t)ir * S.rest_bytes);
    const Cell<real> C(dp, fc, lc, omega);
    const double ri = dp->r_min + ((double)ir + 0.5) * dp->dr;
    const double ktd = dp->dt_dth / ri;
    const real kt = (real)ktd;
    real act[4], aa[4];
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) {
        act[dd] = fabs(ctv[dd]) * kt;
        aa[dd] = acr[dd] + act[dd];
    }

    const bool store = S.useful;
    const int lane = S.lane;
    const uint32_t rowoff = (uint32_t)ir * S.row_bytes;
    const uint32_t pb = opaque(S.pair_bytes);
    const uint32_t pairs = rowoff + S.rest_bytes;

    // stage B stores from every lane, periodic images into their own
    // column of the row padding (nothing reads it): no store sits under a
    // lane mask, which keeps the exec-mask branches and their registers out
    // of the row loop
    const real rest = C.rest(fc[0], C.F[0]);
    if (STAGEA) {
        gold[0] = ga[0][lane];
        ga[0][lane] = rest;
    } else {
        bstore(rest, S.fout, S.vos, rowoff);
    }
#pragma unroll
    for (int k = 1; k <= 4; ++k) {
        const real v = (real)speed(k);
        const real rF = C.rho * C.F[k];
        const real rA = rF * C.factor(v), rB = rF * C.Bz;
        const int base = 1 + 8 * (k - 1);
        const real *x = fc + base;
        // azimuthal neighbours of the ring, every lane taking part in the
        // shifts (lanes 0 and 63 take the halo)
        real nt[8];
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const int c = 4 * (k - 1) + dd;
            nt[left_dir(dd)] = from_left_or(H.l[c], x[left_dir(dd)]);
            nt[right_dir(dd)] = from_right_or(H.r[c], x[right_dir(dd)]);
        }
        if constexpr (MIXED) {
            // from the octant beside: the next direction (left), the one before (right)
            const real s5 = from_left(x[5]), s4 = from_right(x[4]);
            const real l1 = S.turn_left ? nt[2] : nt[1], l2 = S.turn_left ? nt[3] : nt[2];
            const real l3 = S.turn_left ? nt[4] : nt[3], l4 = S.turn_left ? s5 : nt[4];
            const real r5 = S.turn_right ? s4 : nt[5], r6 = S.turn_right ? nt[5] : nt[6];
            const real r7 = S.turn_right ? nt[6] : nt[7], r0 = S.turn_right ? nt[7] : nt[0];
            nt[0] = r0;
            nt[1] = l1;
            nt[2] = l2;
            nt[3] = l3;
            nt[4] = l4;
            nt[5] = r5;
            nt[6] = r6;
            nt[7] = r7;
        }
        real o[8];
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            real E, O;
            pair_coll(C.EP, v * C.EP.w(dd), rA, rB, E, O);
            const real s = C.stay(v, aa[dd]);
            const int c = 4 * (k - 1) + dd;
            constexpr int LOW3 = low_dir(3);
            const int lo = dd < 3 ? dd : LOW3, hi = dd < 3 ? dd + 4 : dd;  // from below, from above
            const real back = behind[c][lane];
            behind[c][lane] = x[lo];
            real ahead;
            if constexpr (STAGEA)
                ahead = fn[base + hi];
            else
                ahead = ga[base + hi][lane];
            o[lo] = dir_new(lo == dd ? E + O : E - O, s, x[lo], v, acr[dd], act[dd], back, nt[lo]);
            o[hi] = dir_new(hi == dd ? E + O : E - O, s, x[hi], v, acr[dd], act[dd], ahead, nt[hi]);
        }
        if (STAGEA) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                gold[base + i] = ga[base + i][lane];
                ga[base + i][lane] = o[i];
            }
        } else {
#pragma unroll
            for (int dd = 0; dd < 4; ++dd)
                bstore2(o[dd], o[dd + 4], S.fout, S.vos2, pairs + (uint32_t)(4 * (k - 1) + dd) * pb);
        }
    }

    const double urp = C.ur(cs), utp = C.ut(cs);
    const double lleft = from_left_or(H.ll, lc);
    const double lright = from_right_or(H.lr, lc);
    const double lr = urp >= 0.0 ? lbehind : lahead;
    const double lt = utp >= 0.0 ? lleft : lright;
    const double lnew = C.lambda(dp, lc, urp, utp, dp->dt_dr, ktd, lr, lt);
    if (STAGEA)
        lout = lnew;
    else
        bstore(lnew, S.lout, S.vols, (uint32_t)ir * S.lrow_bytes);

    if (diag)
        D.add(store, (double)C.rho, (double)C.ux, (double)C.uy, C.Td, (double)C.e, lc, ri * dp->dr * dp->dth, dp->Q);
}

// The intermediate state at the columns bordering strip `strip`, c0 - 1
// (left) and c0 + 64 (right) as periodic images, for the rows [i0, i1) of the
// block, on both sides or on side `only` (every lane then works on that one:
// no more cells are gathered).  LPC lanes (2, or 4 for blocks of at most 8 rows) take one cell:
// lane 32 side + LPC e + h takes row i0 + e of its side and the speeds
// 4 h / LPC + 1 .. 4 (h + 1) / LPC (h = 0 also the rest particle).  Of each
// opposite pair of directions only the one that lane 0 (left side) or lane
// 63 (right side) takes from there is kept.  Each lane gathers its pairs of
// the cell (one access per pair) and, for the kept direction of each, its
// two upwind neighbours (radial ghost rules of Sec. II.D included), which
// side they are on following from the direction alone; the lanes of a cell
// add up their partial moments, and each updates its kept directions as stage
// A of the strip owning the column does, to the same bits.
template <typename real, bool TAUF, int LPC, bool MIXED>
__device__ __forceinline__ void edge_cells(const Strip<real, MIXED> &S, int strip, int i0, int i1,
                                           real (*ef)[FUSE_ROWS][16], double (*el)[FUSE_ROWS], int only)
{
    static_assert(LPC == 2 || LPC == 4, "two or four lanes per cell");
    constexpr int NP = 16 / LPC;  // pairs per lane
    constexpr int NS = 4 / LPC;   // speeds per lane
    const DescPtr dp = S.dp;
    const int lane = S.lane, side = only < 0 ? lane >> 5 : only, e = (lane & 31) / LPC, h = lane & (LPC - 1);
    const int count = i1 - i0;
    const int r = i0 + min(e, count - 1);  // lanes past the block repeat its last row
    const RowBytes rb{S.row_bytes, S.lrow_bytes, S.rest_bytes, S.pair_bytes};
    // the cell, its radial neighbours (below row 0 the copy of row 0, or at
    // a disc centre row 0 with its directions turned by 4; above row nr - 1
    // the copy of row nr - 1) and its azimuthal neighbours
    const EdgeOffsets o = edge_offsets(S.turns, dp->inv2, dp->nr, dp->nt, (int)sizeof(real), rb, strip, side, r);
    const bool turn = dp->disc && r == 0;

    // this lane's pairs NP h .. NP h + NP - 1: directions dd of pair i in
    // x[i], dd + 4 in x[i + NP].  Of each pair only one direction is kept
    // (dd + 4 where `second`), so only its upwind neighbours are gathered.
    real x[2 * NP], nbr[NP], nbt[NP], x0;
    bool second[4];
    bload(x0, S.fin, o.x0, 0u);
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) {
        // the cell's direction dd is direction dd - tc of lane 0 or 63, which
        // takes 1 to 4 from the left, 5, 6, 7, 0 from the right
        const int own = (dd - o.tc) & 7;
        second[dd] = (own >= 1 && own <= 4) == (side == 1);
        const int dir = second[dd] ? dd + 4 : dd;
        const bool low = (dd < 3) != second[dd], left = (dd >= 1) != second[dd];
        // the member of the pair holding the neighbour's value (below the
        // disc centre the opposite direction)
        const int dt = (dir + (left ? o.tl : o.tr)) & 7;
        const uint32_t mr = ((dir >> 2) != (low && turn ? 1 : 0)) ? (uint32_t)sizeof(real) : 0u;
        const uint32_t orad = (low ? o.olo : o.ohi) + o.cc + mr;
        const uint32_t oazi = o.orow + (left ? o.cl : o.cr) + (dt >> 2) * (uint32_t)sizeof(real);
#pragma unroll
        for (int kk = 0; kk < NS; ++kk) {
            const int i = 4 * kk + dd, ring = 4 * (NS * h + kk);
            bload2(x[i], x[i + NP], S.fin, o.orow + o.cc + pair_in_row(rb, ring + dd), 0u);
            bload(nbr[i], S.fin, orad + pair_in_row(rb, ring + dd), 0u);
            bload(nbt[i], S.fin, oazi + pair_in_row(rb, ring + (dt & 3)), 0u);
        }
    }
    double lc, lb, la, lL, lR;
    bload(lc, S.lin, o.lc, 0u);
    bload(lb, S.lin, o.lb, 0u);
    bload(la, S.lin, o.la, 0u);
    bload(lL, S.lin, o.lL, 0u);
    bload(lR, S.lin, o.lR, 0u);
    const double2 cs = dp->cs[o.pc];
    const Polar<real> V(cs);

    real vk[NS];  // this lane's speeds
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
        if constexpr (LPC == 2)
            vk[kk] = h == 0 ? (real)speed(1 + kk) : (real)speed(3 + kk);
        else
            vk[kk] = h == 0 ? (real)speed(1) : h == 1 ? (real)speed(2) : h == 2 ? (real)speed(3) : (real)speed(4);
    }
    real xr[NS][8];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        xr[i >> 2][i & 3] = x[i];
        xr[i >> 2][(i & 3) + 4] = x[i + NP];
    }
    Cell<real> C;
    real jx, jy;
    cell_moments<LPC>(xr, x0, vk, h, C.rho, jx, jy, C.e);
    C.init_moments(dp, jx, jy, lc, omega_at<real, TAUF>(dp, o.om, 0u));

    const double ri = dp->r_min + ((double)r + 0.5) * dp->dr;
    const double ktd = dp->dt_dth / ri;
    const real kr = (real)dp->dt_dr, kt = (real)ktd;
    real g[NP];
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
        const real v = vk[kk];
        real Fk;
        if constexpr (LPC == 2)
            Fk = h == 0 ? C.F[1 + kk] : C.F[3 + kk];
        else
            Fk = h == 0 ? C.F[1] : h == 1 ? C.F[2] : h == 2 ? C.F[3] : C.F[4];
        const real rF = C.rho * Fk;
        const real rA = rF * C.factor(v), rB = rF * C.Bz;
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const int i = 4 * kk + dd;
            const real acr = fabs(V.r[dd]) * kr, act = fabs(V.t[dd]) * kt;
            real E, O;
            pair_coll(C.EP, v * C.EP.w(dd), rA, rB, E, O);
            g[i] = dir_new(second[dd] ? E - O : E + O, C.stay(v, acr + act), second[dd] ? x[i + NP] : x[i], v, acr, act,
                           nbr[i], nbt[i]);
        }
    }
    const double urp = C.ur(cs), utp = C.ut(cs);
    const double lnew =
        C.lambda(dp, lc, urp, utp, dp->dt_dr, ktd, urp >= 0.0 ? lb : la, utp >= 0.0 ? lL : lR);
    // in the order of lane 0's or 63's own pairs (the rows past a short
    // block's last have room here too; a cell's lanes agree on lambda)
#pragma unroll
    for (int i = 0; i < NP; ++i) ef[side][e][NP * h + (i & ~3) + ((i - o.tc) & 3)] = g[i];
    el[side][e] = lnew;
}

// Orders this wavefront's LDS writes before its reads of what other lanes
// wrote (a wavefront's LDS operations complete in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Fills the compact slots of the row behind (see stage_row) from a full row
// x(q), its directions turned by 4 where `turn` (the disc centre's ghost).
template <typename real, class Row>
__device__ __forceinline__ void fill_behind(real (*behind)[64], Row x, bool turn, int lane)
{
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int dd = 0; dd < 4; ++dd) {
            const int lo = dd < 3 ? dd : low_dir(3);
            behind[4 * k + dd][lane] = turn ? x(1 + 8 * k + (lo ^ 4)) : x(1 + 8 * k + lo);
        }
}

// Exchanges two float32 rows of f in registers at the end of a pass.
// Written as plain copies, the loop-carried exchange became three moves per
// value (through a temporary, in three places of the loop); one v_swap_b32
// per value does it (33 instructions instead of 99 per pass).  The s_nop
// gives the two wait states a DPP read of a VGPR needs after a VALU write of
// it, which the compiler does not insert after inline asm.
__device__ __forceinline__ void swap_rows(float (&a)[NQ], float (&b)[NQ])
{
#pragma unroll
    for (int q = 0; q < NQ; ++q) asm("v_swap_b32 %0, %1" : "+v"(a[q]), "+v"(b[q]));
    asm volatile("s_nop 1");
}

// The wavefronts of the workgroup that march the strips beside this one's (w)
// over the same rows: to the left and to the right (-1: in another
// workgroup), and how many rows of g each wavefront has handed on.
struct Beside {
    int w, l, r;
    int *done;
};

// Waits until a wavefront beside has handed on `rows` rows.  It is in the
// same workgroup, so resident, and waits itself only for rows before that.
// LDS carries out a wavefront's operations in order, so what was written
// before the count is there once the count is.
__device__ __forceinline__ void await(int &done, int rows)
{
    while (__builtin_amdgcn_readfirstlane(
               __hip_atomic_load(&done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < rows)
        __builtin_amdgcn_s_sleep(1);
    wave_lds_sync();
}

// Work of one wavefront of the two-step kernel: strip `strip`, rows [i0, i1)
// (at most FUSE_ROWS), marched outward.  Positions p count rows from the
// first row of the block (p = 0); stage A runs on positions -1 .. R where
// they are grid rows, stage B on 0 .. R - 1, one position behind stage A.
// (Odd blocks marched inward read the rows between two blocks at the same
// time as the block beside, 12 % less traffic in float32.  With the sides
// selected at run time that was 1 % faster in float64 and 3 % in float32
// than selecting them for outward marches alone, far less than the selects
// cost; with a march compiled for each direction, 113 KB of code, float64
// took 132 us instead of 126 per 1024 x 1024 launch, float32 79 instead of
// 80, and larger grids 1 to 2 % more: the instruction cache, 64 KB for two
// CUs.)  LDS per wavefront: the
// compact rows behind of f (fb) and of g (gb), the full row of g just
// computed (ga), g at the columns beside the strip (of efs and els, which the
// wavefronts beside write too) and the gathered halo values of stage A's row
// (hb, hbl).
template <typename real, bool TAUF, bool MIXED, class Diag>
__device__ __forceinline__ void march2(DescPtr dp, const StepBufs &bufs, int strip, int i0, int i1,
                                       real (*fb)[64], real (*gb)[64], real (*ga)[64],
                                       real (*efs)[2][FUSE_ROWS][16], double (*els)[2][FUSE_ROWS], real *hb,
                                       double *hbl, const Beside &W, Diag &DA, Diag &DB, bool diagA, bool diagB)
{
    const Strip<real, MIXED> S(dp, bufs, strip);
    const int lane = S.lane;
    const double2 cs = dp->cs[S.pc];
    const Polar<real> V(cs);
    const real kr = (real)dp->dt_dr;
    real acr[4];
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) acr[dd] = fabs(V.r[dd]) * kr;
    const int nr = dp->nr;
    const int count = i1 - i0;
    const bool vlo = i0 > 0, vhi = i1 < nr;  // the rows of positions -1 and R are grid rows

    // f at positions p (fc) and p + 1 (fn) in registers; f(p + 2) is loaded
    // into fc once stage A has used it, and the two swap at the end of the
    // pass.  float64 runs two passes per turn of the loop instead, the second
    // with the roles of the rows exchanged, which takes 130 moves (6 %) off
    // each, 5 us per 1024 x 1024 launch; both copies, 39 KB,
    // still fit the 64 KB instruction cache that two CUs share.  In float32,
    // where the exchange is 33 v_swap_b32, that gained under 1 %.
    real fc[NQ], fn[NQ];
    double lp, lc, ln, lx = 0.0;             // lambda of f at positions p-1, p, p+1, p+2
    double glp = 0.0, glc = 0.0, gln = 0.0;  // lambda of g at positions p-2, p-1, p
    GatherHalo<real> hc, hn, hx;
    int p0;
    real t[NQ];  // the row behind stage A's first row
    auto load_first_rows = [&]() {
        if (vlo) {
            // stage A starts at position -1: behind it position -2 (a ghost
            // beyond the grid), centre -1, ahead 0
            S.load_row(i0 - 1, fc, lc);
            S.load_upwind_halo(i0 - 1, hc.h, hc.hl);
            S.load_row(i0, fn, ln);
            S.load_upwind_halo(i0, hn.h, hn.hl);
            row_or_ghost(S, i0 - 2, t, lp, fc, lc);
            p0 = -1;
        } else {
            S.load_row(i0, fc, lc);
            S.load_upwind_halo(i0, hc.h, hc.hl);
            row_or_ghost(S, i0 + 1, fn, ln, fc, lc);
            if (count > 1 || vhi) S.load_upwind_halo(i0 + 1, hn.h, hn.hl);
            row_or_ghost(S, i0 - 1, t, lp, fc, lc);
            p0 = 0;
        }
    };
    // the edge cells first: issuing the first rows' loads before their
    // gathers, to wait for memory once, took more time in both precisions
    // (97.7 against 95.1 us per float32 launch), the rows held through the
    // edge cells
    // float32 blocks of up to 8 rows: four lanes per edge cell, so that the
    // 2 x 8 cells keep all 64 lanes busy (93.9 against 95.3 us per launch);
    // float64 keeps two (its 16-row blocks fill the lanes with two; with
    // both forms compiled into its kernel it ran 2 us per launch slower)
    real (*ef)[FUSE_ROWS][16] = efs[W.w];
    double (*el)[FUSE_ROWS] = els[W.w];
    const bool hasl = W.l >= 0, hasr = W.r >= 0;
    if (!(hasl && hasr)) {
        const int only = hasl ? 1 : hasr ? 0 : -1;
        if (sizeof(real) == 4 && i1 - i0 <= 8)
            edge_cells<real, TAUF, 4, MIXED>(S, strip, i0, i1, ef, el, only);
        else
            edge_cells<real, TAUF, 2, MIXED>(S, strip, i0, i1, ef, el, only);
    }
    // What this lane hands on of each row of g: lanes 0 to 15 the 16 values
    // that the strip to the left takes from lane 0, lanes 16 to 31 those the
    // strip to the right takes from lane 63, in the order and the frame of
    // edge_cells (the turn is the opposite of this strip's to its neighbour),
    // and lanes 0 and 63 their lambda.  Lanes with nothing to hand on write to
    // their places in hb and hbl, which the next stage A fills anew.
    const int hl = lane >> 4 & 1, hdd = lane & 3;
    const int hdir = ((hl ? left_dir(hdd) : right_dir(hdd)) - (hl ? S.turns.tc[1] : S.turns.tc[0])) & 7;
    const real *hsrc = &ga[1 + 8 * (lane >> 2 & 3) + hdir][hl ? 63 : 0];
    const bool hands = lane < 32 && (hl ? hasr : hasl), handsl = lane == 0 ? hasl : lane == 63 && hasr;
    real *hdst = hands ? &efs[hl ? W.r : W.l][hl ? 0 : 1][0][lane & 15] : hb + lane;
    double *hdstl = handsl ? &els[lane ? W.r : W.l][lane ? 0 : 1][0] : hbl + lane;
    // TAUF: exp(-dt/tau) of stage A's row (oa), loaded a pass ahead, and of
    // stage B's (ob), the row stage A had a pass before (loaded at the point
    // of use, the field cost 7.2 us per float64 launch and 4.2 us per float32
    // one; loaded ahead, 0.8 and 2.3 us)
    real oa = (real)0, ob = (real)0;
    if constexpr (TAUF) oa = omega_at<real, true>(dp, S.vo, (uint32_t)(vlo ? i0 - 1 : i0) * S.rest_bytes);
    load_first_rows();
    fill_behind(fb, [&](int q) { return t[q]; }, false, lane);
    if constexpr (TAUF) settle(oa);
    wave_lds_sync();

    // one pass: stage A at position p (f(p) in fc, f(p + 1) in fn), stage B one behind
    auto pass = [&](int p, real (&fc)[NQ], real (&fn)[NQ]) __attribute__((always_inline)) {
        const int ir = i0 + p;
        // g(p - 1), centre of stage B: stage A hands it over as it replaces
        // it in ga
        real gc[NQ];
        // g(-1), computed by stage A at position -1, is the row behind
        // stage B's first row
        if (p == 0 && vlo) fill_behind(gb, [&](int q) { return ga[q][lane]; }, false, lane);
        // (A) first step at position p, or the ghost beyond the grid
        if (p < count || vhi) {
            // the row's gathered halo values into LDS, read back by every lane
            hb[lane] = hc.h;
            hbl[lane] = hc.hl;
            wave_lds_sync();
            const Halo<real> H{hb, hb + 16, hbl[0], hbl[1]};
            stage_row<real, true, TAUF>(S, ir, fb, fc, fn, ga, gc, H, lp, lc, ln, acr, V.t, cs, gln, oa, DA,
                                        diagA && p >= 0 && p < count);
        } else {
            // beyond the last grid row: the zero-gradient ghost of g
#pragma unroll
            for (int q = 0; q < NQ; ++q) gc[q] = ga[q][lane];
            gln = glc;
        }
        // hand the row's ends on
        if ((hasl || hasr) && p >= 0 && p < count) {
            wave_lds_sync();
            hdst[hands ? p * 16 : 0] = *hsrc;
            hdstl[handsl ? p : 0] = gln;
            wave_lds_sync();
            __hip_atomic_store(&W.done[W.w], p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        // f at position p + 2 (the row ahead of the next stage A) replaces f(p)
        if (p + 1 < count || (p + 1 == count && vhi)) row_or_ghost(S, ir + 2, fc, lx, fn, ln);
        if (p + 2 < count || (p + 2 == count && vhi)) S.load_upwind_halo(ir + 2, hx.h, hx.hl);
        // the next stage A's exp(-dt/tau), where that stage runs on a grid row
        const real oa_used = oa;
        if constexpr (TAUF) {
            if (p + 1 < count || (p + 1 == count && vhi))
                oa = omega_at<real, true>(dp, S.vo, (uint32_t)(ir + 1) * S.rest_bytes);
        }
        // (B) second step at position p - 1
        if (p == 0 && !vlo) {
            // the row behind stage B's first row is the (zero-gradient)
            // ghost of g(0) (at a disc centre with every direction turned by 4)
            fill_behind(gb, [&](int q) { return ga[q][lane]; }, dp->disc, lane);
            glc = gln;
        } else if (p > 0) {
            if (hasl) await(W.done[W.l], p);
            if (hasr) await(W.done[W.r], p);
            const Halo<real> H{ef[0][p - 1], ef[1][p - 1], el[0][p - 1], el[1][p - 1]};
            double unused;
            stage_row<real, false, TAUF>(S, ir - 1, gb, gc, nullptr, ga, nullptr, H, glp, glc, gln, acr, V.t, cs, unused,
                                         ob, DB, diagB);
        }
        ob = oa_used;
        hc = hn;
        hn = hx;
        lp = lc;
        lc = ln;
        ln = lx;
        glp = glc;
        glc = gln;
        // Compiler-only barrier: the LDS rows must not be promoted to
        // registers across passes.
        asm volatile("" ::: "memory");
    };
    if constexpr (sizeof(real) == 8) {
        for (int p = p0; p <= count; p += 2) {
            pass(p, fc, fn);
            if (p + 1 > count) break;
            pass(p + 1, fn, fc);
        }
    } else {
        for (int p = p0; p <= count; ++p) {
            pass(p, fc, fn);
            swap_rows(fc, fn);
        }
    }
}

// Wavefronts per SIMD of the two-step kernel: one in float64, whose two
// steps' rows fill the register file, two in float32.
template <typename real>
struct Step2Occ {
    static constexpr int waves = sizeof(real) == 4 ? 2 : 1;
};

// Steps s and s + 1 of every solve of the launch in one pass over f.  Tiles,
// step bases and step_off as k_step's (a single solve passes no tile table,
// so wavefront t takes its tile t, and no bases, so s = step_off).  The state
// of step s of solve i is in buffer (s + flip_i) & 1 with flip_i = flips[i]
// ^ flip (flips may be NULL); a two-step launch leaves it in the other
// buffer, so the caller toggles flip_i after it.  A solve with one step left,
// or every solve when `single` is set, takes one step instead (the one-step
// march), which keeps the parity.  One wavefront per SIMD in float64, where
// the two steps' rows fill the register file and the LDS rows of four
// wavefronts most of a CU's LDS; two in float32, whose rows take half the
// LDS.  MIXED: grids whose octants are not whole strips (whole_octants).
template <typename real, bool TAUF, bool MIXED>
__global__ __launch_bounds__(BLOCK, Step2Occ<real>::waves) void k_step2(const SolveDesc *descs, const uint2 *tiles,
                                                                       int ntiles, const int64_t *bases,
                                                                       int64_t step_off, const int *flips, int flip,
                                                                       int single)
{
    const int nb = gridDim.x;
    const int blk = xcd_tile(blockIdx.x, nb);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __shared__ int done[BLOCK / 64];
    done[w] = 0;
    __syncthreads();
    const int t = blk * (BLOCK / 64) + w;
    if (t >= ntiles) return;
    int solve = 0, lt = t;
    if (tiles) {
        const uint2 e = tiles[t];
        solve = __builtin_amdgcn_readfirstlane((int)e.x);
        lt = __builtin_amdgcn_readfirstlane((int)e.y);
    }
    const DescPtr dp = (DescPtr)(descs + solve);
    const int64_t step = (bases ? bases[solve] : 0) + step_off;
    if (step >= dp->nsteps) return;
    const int cur = (int)((step + ((flips ? flips[solve] : 0) ^ flip)) & 1);
    const StepBufs bufs{dp->f[cur], dp->f[cur ^ 1], dp->lam[cur], dp->lam[cur ^ 1]};
    __shared__ real fb[BLOCK / 64][16][64];
    __shared__ real gb[BLOCK / 64][16][64];
    __shared__ real ga[BLOCK / 64][NQ][64];
    __shared__ real ef[BLOCK / 64][2][FUSE_ROWS][16];
    __shared__ double el[BLOCK / 64][2][FUSE_ROWS];
    __shared__ real hb[BLOCK / 64][64];
    __shared__ double hbl[BLOCK / 64][64];
    const int rows = dp->rows, nstrip = dp->nstrip;
    const int rb = lt / nstrip, strip = lt - rb * nstrip;
    const int i0 = rb * rows;
    const int i1 = min(i0 + rows, dp->nr);
    if (single || step + 1 >= dp->nsteps) {
        // one step, with the row behind in the LDS row of g
        const bool diag = records(dp, step);
        double red[5] = {0, 0, 0, 0, 0};
        // (odd blocks inward, beside the rows of the block before, in float32
        // alone: 16 packed 300 x 200 then take 88 us, 91 all outward; in
        // float64, 145 and 149, the 16 KB of code cost the pairs more: 20
        // steps of 1024 x 512 took 749 us with them, 741 without)
        if (sizeof(real) == 4 && (rb & 1) != 0)
            march<real, MIXED, TAUF, true>(dp, bufs, strip, i0, i1, ga[w], red, diag);
        else
            march<real, MIXED, TAUF, false>(dp, bufs, strip, i0, i1, ga[w], red, diag);
        if (diag) {
            const int64_t slot = (step / dp->diag_every) % PART_RING;
            double *part = dp->wpart + ((size_t)slot * dp->nwaves + lt) * 5;
            double v[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) v[i] = wave_sum(red[i]);
            if ((threadIdx.x & 63) == 0)
#pragma unroll
                for (int i = 0; i < 5; ++i) part[i] = v[i];
        }
        return;
    }
    const bool diagA = records(dp, step), diagB = records(dp, step + 1);
    LaneDiag DA, DB;
    // the strips beside, where whole strips or more columns follow
    const bool wraps = dp->nt % STRIP == 0;
    const int wl = w + (strip > 0 ? -1 : nstrip - 1), wr = w + (strip < nstrip - 1 ? 1 : 1 - nstrip);
    const Beside W{w, (strip > 0 || wraps) && wl >= 0 && wl < BLOCK / 64 ? wl : -1,
                   (strip < nstrip - 1 || wraps) && wr >= 0 && wr < BLOCK / 64 ? wr : -1, done};
    march2<real, TAUF, MIXED>(dp, bufs, strip, i0, i1, fb[w], gb[w], ga[w], ef, el, hb[w], hbl[w], W,
                            DA, DB, diagA, diagB);
    // both steps' totals first (independent DPP chains the compiler can
    // interleave), then one lane stores them
    double v[2][5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        v[0][i] = diagA ? DA.total(i) : 0.0;
        v[1][i] = diagB ? DB.total(i) : 0.0;
    }
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (!(s == 0 ? diagA : diagB)) continue;
            const int64_t slot = ((step + s) / dp->diag_every) % PART_RING;
            double *part = dp->wpart + ((size_t)slot * dp->nwaves + lt) * 5;
#pragma unroll
            for (int i = 0; i < 5; ++i) part[i] = v[s][i];
            if (!tiles) clear_rest(dp, part, lt, ntiles);
        }
    }
}

}  // namespace

template <typename real, bool TAUF, bool MIXED>
static void launch_k_step2(int nb, hipStream_t st, const SolveDesc *descs, const uint2 *tiles, int ntiles,
                           const int64_t *bases, int64_t step_off, const int *flips, int flip, bool single)
{
    hipLaunchKernelGGL((k_step2<real, TAUF, MIXED>), dim3(nb), dim3(BLOCK), 0, st, descs, tiles, ntiles, bases, step_off,
                       flips, flip, (int)single);
}

hipError_t launch_step2(const SolveDesc *descs, const uint2 *tiles, int ntiles, const int64_t *bases,
                        int64_t step_off, const int *flips, int flip, bool single, bool fp32, bool tauf, bool mixed,
                        hipStream_t st)
{
    const int nb = (ntiles + BLOCK / 64 - 1) / (BLOCK / 64);
    if (nb == 0) return hipSuccess;
    // named in the order in which they are to lie in the code object: the
    // float64 kernels of 72 KB exceed the instruction cache and feel where they
    // start (1024 x 1024, with drift records: 130.4 us this way, 130.8 with the
    // float32 kernels first, at times 130.5 or 131.1 for other code between)
    auto *fn = !fp32 ? (!mixed ? (!tauf ? &launch_k_step2<double, false, false> : &launch_k_step2<double, true, false>)
                               : (!tauf ? &launch_k_step2<double, false, true> : &launch_k_step2<double, true, true>))
                     : (!mixed ? (!tauf ? &launch_k_step2<float, false, false> : &launch_k_step2<float, true, false>)
                               : (!tauf ? &launch_k_step2<float, false, true> : &launch_k_step2<float, true, true>));
    fn(nb, st, descs, tiles, ntiles, bases, step_off, flips, flip, single);
    return hipGetLastError();
}

}  // namespace pdbm
