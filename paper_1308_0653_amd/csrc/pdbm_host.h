// Host-side internals shared by the single-solve, batch and server parts of
// libpdbm.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>
#include <vector>

#include "pdbm_internal.h"
#include "pdbm_offsets.h"

namespace pdbm {

// Records `msg` as the calling thread's last error and returns `code`.
int fail(int code, const std::string &msg);

#define PDBM_HIPCHK(call)                                                                                      \
    do {                                                                                                       \
        hipError_t e_ = (call);                                                                                \
        if (e_ != hipSuccess) return ::pdbm::fail(PDBM_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

// Device memory of one solve, in this order (all offsets 256-byte aligned):
// the state (two f buffers, two lambda buffers, the per-cell relaxation
// factors of a solve with PDBM_TAU_FIELD), then the auxiliary part
// (theta table, description, step state, drift partial sums and records,
// moments reduction scratch).
struct Layout {
    size_t f, lam, omega, cs, desc, state, wpart, hist, cpart, total;  // omega: per-cell relaxation factors (0 without PDBM_TAU_FIELD)
    size_t state_total, aux_total;  // total = state_total + aux_total
    int pitch, rows, nwaves, cblocks;
    size_t esz;
};

// `rows`: rows per wavefront of the marching kernels, or PATCHES for a solve
// stepped on patches (patch_geom).
constexpr int PATCHES = 0;

// How long a launch of this many wavefronts takes, in the times one of them
// takes on a full GPU (1024 SIMDs; one wavefront on each in float64, two in
// float32, where one alone runs faster, and memory serves fewer of them
// faster).  From timings of 300 x 380 to 3000 x 1024 grids and packs of 1 to
// 40 in blocks of 2 to 16 rows: the wavefronts of a last round that is not
// full take 0.6 of its time longer than their share (0.4 in float32).
inline double launch_rounds(int64_t waves, bool fp32)
{
    const double x = (double)waves / (fp32 ? 2048 : 1024);
    if (fp32 && x <= 0.5) return 0.55 + 0.25 * x;
    if (x <= 1.0) return fp32 ? 0.6 + 0.4 * x : 1.0;
    return x + (fp32 ? 0.4 : 0.6) * (std::ceil(x) - x);
}
// Rows per wavefront of the marching kernels for a launch of waves(r)
// wavefronts in blocks of r rows: long blocks compute and read the fewest
// rows twice, but a wavefront of r rows takes about the time of r + more
// (a pair of steps 2 r + 5 rows, both steps' and the two beside the block and
// its start, MORE_PAIR; a single step r + 2), whole rounds of which make the
// launch.  Between FEWEST_ROWS and FUSE_ROWS rows, more than `most`
// wavefronts only where FUSE_ROWS needs them.  With the fewest rows that make
// one round, else 16, 1100 x 1024 took 220 us per two steps in float64 and
// takes 161 (1.92 rounds of 9 rows instead of 1.08 of 16), 1500 x 1024 229
// and 200; in float32 2400 x 1024 207 and 182, 1280 x 1800 217 and 187.
constexpr int FEWEST_ROWS = 2;
constexpr double MORE_PAIR = 2.5, MORE_SINGLE = 2.0;
template <class Waves>
int best_rows(Waves waves, bool fp32, int64_t most, double more = MORE_PAIR)
{
    int best = FUSE_ROWS;
    double least = 0.0;
    for (int r = FUSE_ROWS; r >= FEWEST_ROWS; --r) {
        const int64_t n = waves(r);
        if (r < FUSE_ROWS && n > most) break;
        const double t = (r + more) * launch_rounds(n, fp32);
        if (r == FUSE_ROWS || t < least) {
            best = r;
            least = t;
        }
    }
    return best;
}

Layout layout_of(const pdbm_params &p, int rows, bool alone);
// Rows per wavefront a packed solve starts with, or PATCHES (Pack::rebuild
// chooses them anew with every change of the pack, unless PDBM_BATCH_ROWS
// fixes them).
int batch_rows(const pdbm_params &p);
int batch_rows_env();
// Rows per wavefront of the one-step launches of such a solve, or PATCHES.
int rows_one(const pdbm_params &p, int rows, bool alone);
// Patches of a solve that rows_per_wave (alone) or batch_rows gives them.
PatchGeom patches(const pdbm_params &p, bool alone);
class Solve;
// Non-equilibrium measures of the current state into host `out`
// [NONEQ][nr][ntheta] (staged in the idle f buffer; synchronises st).
int noneq_to_host(const Solve &s, double *out, hipStream_t st);
int check_device();

// One solve resident on the GPU: its buffers, the description its kernels
// read and a host mirror of its step counter.
class Solve {
  public:
    pdbm_params p{};
    Layout L{};
    bool fp32 = false, own = false;
    char *ws = nullptr;
    SolveDesc hd{};           // host copy, pointers filled in
    SolveDesc *dd = nullptr;  // device copy read by the step kernel
    double *cpart = nullptr;  // moments-kernel reduction scratch
    int64_t step = 0;      // steps taken (never beyond hd.nsteps)
    int flip = 0;          // the current state is in buffer (step + flip) & 1 (two-step launches toggle it)
    int64_t rec_from = 0;  // drift records are valid from this step on
    int64_t red_to = 0;    // records of steps before this one have been added up
    SolveState zero_state{};  // staging of the step-state upload (kept until the next sync)

    // Lays out the solve in `workspace` (or a fresh allocation), uploads its
    // description and enqueues its initial state on `st`.  `rows`: rows per
    // wavefront or PATCHES; `nsteps`: step count after which the solve stops
    // advancing; `alone`: it has the GPU to itself (no pack).
    // With `aux`, the workspace holds the state only (L.state_total bytes)
    // and the auxiliary part goes to `aux` (L.aux_total bytes, 256-byte
    // aligned).  Allocates device memory only when workspace is NULL and no
    // host memory at all.
    int init(const pdbm_params &p, const pdbm_ic *ic, void *workspace, size_t bytes, int rows, int64_t nsteps,
             bool alone, hipStream_t st, char *aux = nullptr);
    void release();  // frees an owned workspace (the stream must be idle)

    int cur() const { return (int)((step + flip) & 1); }
    // Whether two steps may go in one launch: ntheta > 1 and row blocks of
    // at most FUSE_ROWS rows, not stepped on patches (either precision, any
    // sector; PDBM_FUSE=0 turns it off).
    bool fusable() const;
    // Whether a launch may take up to COL_K steps: a single theta column
    // (PDBM_FUSE=0 turns it off: one step per launch, k_step).
    bool columnar() const;
    // Whether its launches step patches of the grid, up to geom.k steps each.
    bool patched() const { return hd.patch.threads > 0; }
    int patch_steps() const;  // ... of this many steps at most
    // Wavefronts or patches of its launches, and wavefronts of those that
    // march a single step.
    int waves() const { return patched() ? hd.patch.ntiles : solve_waves(p.nr, p.ntheta, hd.rows); }
    int waves_one() const { return solve_waves(p.nr, p.ntheta, hd.rows1); }
    // Marches blocks of `rows` rows from now on (a member of a pack).  A
    // solve that makes drift records keeps the blocks it has memory for the
    // partial sums of.
    void set_rows(int rows)
    {
        hd.rows = hd.rows1 = p.diag_every > 0 ? L.rows : rows;
        hd.nwaves = waves_at(rows);
    }
    int waves_at(int rows) const { return solve_waves(p.nr, p.ntheta, p.diag_every > 0 ? L.rows : rows); }
    bool mixed() const { return !whole_octants(p.ntheta, p.sector); }
    bool tauf() const { return hd.omegaf != nullptr; }  // relaxes with a per-cell tau
    // Sets the step count on host and device (stream must be idle).
    int set_step(int64_t s, hipStream_t st);
    // Enqueues the adding up of the drift partial sums of steps [red_to,
    // step), at most PART_RING steps (single-solve launches only).
    int reduce_records(hipStream_t st);
    // Fields [6][nr][ntheta] of the current state into device memory `out`
    // and the drift report into `diag_dev` (both enqueued on st).
    int moments(double *out, pdbm_diag *diag_dev, hipStream_t st) const;
};

// Ends a solver made by pdbm_create_noalloc: frees its device's static
// scratch for the next one (pdbm_noalloc.hip).
void release_scratch_solver(int dev);

}  // namespace pdbm

// Handle of one solve (the opaque pdbm_solver of the ABI).
struct pdbm_solver {
    pdbm::Solve s;
    hipStream_t st = nullptr;
    int scratch_dev = -1;  // device whose static scratch holds the auxiliary part (pdbm_create_noalloc), or -1
};
