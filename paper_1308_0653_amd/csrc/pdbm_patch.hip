// Several time steps per launch on patches of a small grid (k_patch): grids
// too small to fill the GPU with wavefronts that march along r, where a step
// takes as long as one wavefront's serial chain of instructions.
#include "pdbm_device.h"

namespace pdbm {
namespace {

// A workgroup holds one patch of the grid with a halo of g.k rows and
// columns (patch_cell) and takes up to g.k steps of it; after each step the
// cells one further in from the edge of the halo still hold the true state,
// and after the last its own cells, which it stores.  Workgroups never wait
// for one another.
//
// Two or four lanes (LPC) take a cell, lane h the rings of speeds 4 h / LPC + 1
// to 4 (h + 1) / LPC (lane 0 also the rest particle): each keeps its rings'
// distributions in registers, they add up their partial moments (DPP), and each
// updates its rings, so the chain of a cell's step is about a half or a quarter
// of what one lane would run.
// The upwind neighbours come from LDS, where every cell publishes its
// distributions at the start of a step in one of two buffers (one barrier
// per step): element (direction d, thread t) at d * threads + t, so that
// adjacent lanes read adjacent elements.  A lane's sixteen neighbour
// addresses are the same in every step: they carry the side that is upwind
// for the direction, the radial ghosts of Sec. II.D (a cell's own value, at a
// disc centre that of the opposite direction), the turn of the directions
// between columns of different octants and, on a patch that holds the whole
// ring, its closing.
template <typename real, bool TAUF, int LPC, int NT>
__global__ __launch_bounds__(NT, 1) void k_patch(const SolveDesc *descs, const uint2 *tiles, const int64_t *bases,
                                                 int64_t step_off, const int *flips, int flip, int nk_most)
{
    static_assert(LPC == 2 || LPC == 4, "two or four lanes per cell");
    constexpr int NS = 4 / LPC;  // rings per lane
    __shared__ real planes[2][NS * 8][NT];
    __shared__ double lams[2][NT / LPC];
    __shared__ double parts[2][NT / 64][5];
    const int t = threadIdx.x, h = t & (LPC - 1);
    int tile = xcd_tile(blockIdx.x, gridDim.x), solve = 0;
    if (tiles) {
        const uint2 e = tiles[tile];
        solve = __builtin_amdgcn_readfirstlane((int)e.x);
        tile = __builtin_amdgcn_readfirstlane((int)e.y);
    }
    const DescPtr dp = (DescPtr)(descs + solve);
    const int64_t step0 = (bases ? bases[solve] : 0) + step_off;
    if (step0 >= dp->nsteps) return;
    const int nk = (int)min((int64_t)nk_most, dp->nsteps - step0);
    const PatchGeom g{dp->patch.rows, dp->patch.cols, dp->patch.k, dp->patch.nbc, dp->patch.ntiles, NT, LPC};
    const int nr = dp->nr, nt = dp->nt;
    const int cur = (int)((step0 + ((flips ? flips[solve] : 0) ^ flip)) & 1);
    const __amdgpu_buffer_rsrc_t fin = rsrc_of(dp->f[cur]), fout = rsrc_of(dp->f[cur ^ 1]);
    const __amdgpu_buffer_rsrc_t lin = rsrc_of(dp->lam[cur]), lout = rsrc_of(dp->lam[cur ^ 1]);
    const RowBytes b = row_bytes_of(dp->rstride, dp->pitch, (int)sizeof(real));
    const PatchCell c = patch_cell(g, nr, nt, dp->inv2, tile, t / LPC);

    // the state at step0: this lane's ring, the rest particle, lambda
    const PatchOffsets o = patch_offsets(c, b, (int)sizeof(real), LPC, h);
    real x[NS][8], x0;
    double lc;
#pragma unroll
    for (int i = 0; i < 4 * NS; ++i) bload2(x[i >> 2][i & 3], x[i >> 2][(i & 3) + 4], fin, o.pair, (uint32_t)i * b.pair);
    bload(x0, fin, o.rest, 0u);
    bload(lc, lin, o.lam, 0u);
    const real om = omega_at<real, TAUF>(dp, o.om, 0u);
    // this ring's row of the moment inversion, read again in every step
    __shared__ double Arow[16];
    if (t < 16) Arow[t] = dp->A[t];
    __syncthreads();
    real v[NS];
#pragma unroll
    for (int kk = 0; kk < NS; ++kk) {
        if constexpr (LPC == 4)
            v[kk] = h == 0 ? (real)speed(1) : h == 1 ? (real)speed(2) : h == 2 ? (real)speed(3) : (real)speed(4);
        else
            v[kk] = h == 0 ? (real)speed(1 + kk) : (real)speed(3 + kk);
    }

    const double2 cs = dp->cs[c.pc];
    const double ri = dp->r_min + ((double)c.row + 0.5) * dp->dr;
    const double ktd = dp->dt_dth / ri;
    const real kr = (real)dp->dt_dr, kt = (real)ktd;
    // elements of the upwind neighbours: below for directions 0, 1, 2 and 7
    // (from this many planes on), above for 3 to 6, left and right by pair
    const PatchNear near = patch_near(c, dp->inv2, nt, dp->sector, t / LPC);
    const int turned = c.row == 0 && dp->disc ? 4 * NT : 0;
    const int low = near.low * LPC + h + turned, low7 = near.low * LPC + h - turned, high = near.high * LPC + h;
    int left[4], right[4];
#pragma unroll
    for (int dd = 0; dd < 4; ++dd) {
        left[dd] = ((left_dir(dd) + near.turn_left) & 7) * NT + near.left * LPC + h;
        right[dd] = ((right_dir(dd) + near.turn_right) & 7) * NT + near.right * LPC + h;
    }
    const int spare = g.k - nk;  // halo not used up by a launch of fewer steps

    for (int j = 0; j < nk; ++j) {
        const int64_t step = step0 + j;
        real *const P = planes[j & 1][0];
        double *const Lm = lams[j & 1];
        double(*const part)[5] = parts[j & 1];
        const bool rec = records(dp, step);
        // a wavefront all of whose cells are used up takes no further part
        const bool publish = __builtin_amdgcn_ballot_w64(c.dist >= j + spare) != 0;
        const bool update = __builtin_amdgcn_ballot_w64(c.dist > j + spare) != 0;
        Cell<real> C;
        real Fk[NS] = {}, F0 = 0;
        if (publish) {
#pragma unroll
            for (int i = 0; i < 8 * NS; ++i) P[i * NT + t] = x[i >> 3][i & 7];
            Lm[t / LPC] = lc;  // the same from each of a cell's lanes
        }
        if (update) {
            real jx, jy;
            cell_moments<LPC>(x, x0, v, h, C.rho, jx, jy, C.e);
            C.init_state(dp, jx, jy, lc, om);
            const double T2 = C.Td * C.Td, T3 = T2 * C.Td, T4 = T2 * T2;
            double sum = 0.0;
#pragma unroll
            for (int kk = 0; kk < NS; ++kk) {
                const double *A = Arow + 4 * (NS * h + kk);
                const double F = fma(A[3], T4, fma(A[2], T3, fma(A[1], T2, A[0] * C.Td)));
                Fk[kk] = (real)F;
                sum = kk > 0 ? sum + F : F;
            }
            F0 = (real)fma(-8.0, cell_sum<LPC>(sum), 1.0);
        }
        if (rec) {
            double red[5] = {0, 0, 0, 0, 0};
            if (update)
                diag_cell(red, c.own && h == 0, (double)C.rho, (double)C.ux, (double)C.uy, C.Td, (double)C.e, lc,
                          (dp->r_min + ((double)c.row + 0.5) * dp->dr) * dp->dr * dp->dth, dp->Q);
            double s[5];
#pragma unroll
            for (int i = 0; i < 5; ++i) s[i] = wave_sum(red[i]);
            if ((t & 63) == 0)
#pragma unroll
                for (int i = 0; i < 5; ++i) part[t >> 6][i] = s[i];
        }
        __syncthreads();
        if (rec && t == 0) {
            double *out = dp->wpart + (((size_t)((step / dp->diag_every) % PART_RING)) * dp->nwaves + tile) * 5;
            // (of 12 wavefronts and two lanes to a cell all at once they spill
            // to scratch memory; one at a time of 4 wavefronts, 400 steps of a
            // 20000-row column took 3 % longer)
            constexpr int AT_ONCE = NT > 512 && LPC == 2 ? 1 : 5;
#pragma unroll AT_ONCE
            for (int i = 0; i < 5; ++i) {
                double s = part[0][i];
                for (int w = 1; w < NT / 64; ++w) s += part[w][i];
                out[i] = s;
            }
            if constexpr (marched_beside(LPC)) {
                if (!tiles) clear_rest(dp, out, tile, g.ntiles);
            }
        }
        if (update) {
            // worked out again in every step, which takes fewer registers
            double2 a = cs;
            asm volatile("" : "+v"(a.x), "+v"(a.y));
            const Polar<real> V(a);
            real acr[4], act[4];
#pragma unroll
            for (int dd = 0; dd < 4; ++dd) {
                acr[dd] = fabs(V.r[dd]) * kr;
                act[dd] = fabs(V.t[dd]) * kt;
            }
#pragma unroll
            for (int kk = 0; kk < NS; ++kk) {
                const real *Pk = P + kk * 8 * NT;
                const real rF = C.rho * Fk[kk];
                const real rA = rF * C.factor(v[kk]), rB = rF * C.Bz;
#pragma unroll
                for (int dd = 0; dd < 4; ++dd) {
                    real E, O;
                    pair_coll(C.EP, v[kk] * C.EP.w(dd), rA, rB, E, O);
                    const real s = C.stay(v[kk], acr[dd] + act[dd]);
                    const real rad0 = Pk[dd * NT + (dd < 3 ? low : high)];
                    const real rad4 = Pk[(dd + 4) * NT + (dd < 3 ? high : low7)];
                    const real azi0 = Pk[dd > 0 ? left[dd] : right[dd]], azi4 = Pk[dd > 0 ? right[dd] : left[dd]];
                    const real o0 = dir_new(E + O, s, x[kk][dd], v[kk], acr[dd], act[dd], rad0, azi0);
                    x[kk][dd + 4] = dir_new(E - O, s, x[kk][dd + 4], v[kk], acr[dd], act[dd], rad4, azi4);
                    x[kk][dd] = o0;
                }
            }
            x0 = C.rest(x0, F0);
            // lambda: closed-form Cochran step, then upwind by own-cell u
            const double urp = C.ur(cs), utp = C.ut(cs);
            const double lr = Lm[urp >= 0.0 ? near.low : near.high];
            const double lt = Lm[utp >= 0.0 ? near.left : near.right];
            lc = C.lambda(dp, lc, urp, utp, dp->dt_dr, ktd, lr, lt);
        }
    }

    if (c.own) {
#pragma unroll
        for (int i = 0; i < 4 * NS; ++i)
            bstore2(x[i >> 2][i & 3], x[i >> 2][(i & 3) + 4], fout, o.pair, (uint32_t)i * b.pair);
        if (h == 0) {
            bstore(x0, fout, o.rest, 0u);
            bstore(lc, lout, o.lam, 0u);
        }
    }
}

}  // namespace

// A kernel per precision and tau field for the lanes per cell and the
// workgroup sizes that the shapes of pdbm_offsets.h use.
template <typename real, bool TAUF>
static auto patch_kernel(int threads, int lanes) -> decltype(&k_patch<real, TAUF, 2, 512>)
{
    constexpr bool fp32 = sizeof(real) == 4;
    switch (8 * threads + lanes) {
    case 8 * 256 + 2: return &k_patch<real, TAUF, 2, 256>;
    case 8 * 256 + 4: return &k_patch<real, TAUF, 4, 256>;
    case 8 * 512 + 2: return &k_patch<real, TAUF, 2, 512>;
    case 8 * 512 + 4:
        if constexpr (!fp32) return &k_patch<real, TAUF, 4, 512>;
        break;
    case 8 * 768 + 2:
        if constexpr (fp32) return &k_patch<real, TAUF, 2, 768>;  // (200 KB of LDS in float64)
        break;
    case 8 * 768 + 4:
        if constexpr (fp32) return &k_patch<real, TAUF, 4, 768>;
        break;
    }
    return nullptr;
}

hipError_t launch_patch(const SolveDesc *descs, const uint2 *tiles, int ntiles, int threads, int lanes,
                        const int64_t *bases, int64_t step_off, const int *flips, int flip, int nk, bool fp32, bool tauf,
                        hipStream_t st)
{
    if (ntiles == 0 || nk <= 0) return hipSuccess;
    auto *fn = fp32 ? (tauf ? patch_kernel<float, true>(threads, lanes) : patch_kernel<float, false>(threads, lanes))
                    : (tauf ? patch_kernel<double, true>(threads, lanes) : patch_kernel<double, false>(threads, lanes));
    if (!fn) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fn, dim3(ntiles), dim3(threads), 0, st, descs, tiles, bases, step_off, flips, flip, nk);
    return hipGetLastError();
}

}  // namespace pdbm
