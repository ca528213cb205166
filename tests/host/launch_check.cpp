// CPU check of the launches that pdbm_step makes of single solves, on the
// model GPU of model_gpu.h: how many steps each takes, in which kernel, of how
// many wavefronts or patches; and of the copies that reading the raw state
// takes.  Exit status 0 when every check holds.
#include "model_gpu.h"

namespace {

int fails = 0;

// The launches of one call of `steps` steps, as "kernel steps x tiles" each.
void call(int nr, int nt, int precision, int steps, const std::string &want, bool captured = false)
{
    pdbm_params p{};
    p.nr = nr;
    p.ntheta = nt;
    p.sector = 8;
    p.precision = precision;
    p.diag_every = 1;
    p.r_min = 0.3;
    p.r_max = 1.0;
    p.dt = 1e-9;
    p.tau = 1e-3;
    hipStream_t st = nullptr;
    (void)hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    pdbm_solver *s = nullptr;
    std::string got;
    if (pdbm_create(&p, nullptr, nullptr, 0, st, &s) == PDBM_OK) {
        gpu.log.clear();
        gpu.logging = true;
        if (captured) gpu.capturing = (void *)st;
        (void)pdbm_step(s, steps);
        gpu.capturing = nullptr;
        gpu.logging = false;
        for (const auto &l : gpu.log)
            got += (got.empty() ? "" : " ") + std::string(1, l.kernel) + std::to_string(l.steps) + "x" + std::to_string(l.tiles);
        pdbm_destroy(s);
    }
    (void)hipStreamDestroy(st);
    if (got != want) {
        std::fprintf(stderr, "FAILED %d x %d precision %d, %d steps: %s, not %s\n", nr, nt, precision, steps, got.c_str(),
                     want.c_str());
        fails++;
    }
}

// Copies of one read of f and lambda.
void reads(int nr, int nt, int precision, int want)
{
    pdbm_params p{};
    p.nr = nr;
    p.ntheta = nt;
    p.sector = 8;
    p.precision = precision;
    p.r_min = 0.3;
    p.r_max = 1.0;
    p.dt = 1e-9;
    p.tau = 1e-3;
    pdbm_solver *s = nullptr;
    std::vector<double> f((size_t)33 * nr * nt), lam((size_t)nr * nt);
    if (pdbm_create(&p, nullptr, nullptr, 0, nullptr, &s) == PDBM_OK) {
        gpu.copies = 0;
        gpu.logging = true;
        (void)pdbm_read_f(s, f.data(), lam.data());
        gpu.logging = false;
        pdbm_destroy(s);
    }
    if (gpu.copies != want) {
        std::fprintf(stderr, "FAILED read of %d x %d precision %d: %d copies, not %d\n", nr, nt, precision, gpu.copies, want);
        fails++;
    }
}

}  // namespace

int main()
{
    // lambda, and f at once: in its own precision, or as much of it in float64 as the idle buffer holds
    reads(64, 64, PDBM_FP64, 2);
    reads(8, 64, PDBM_FP32, 2);
    reads(32, 64, PDBM_FP32, 2);
    reads(33, 64, PDBM_FP32, 4);
    reads(400, 20, PDBM_FP32, 2);
    reads(100, 100, PDBM_FP32, 3);
    // on patches, single steps too up to two rounds of them (260 x 260: 484 of 12 x 12 cells) ...
    call(64, 64, PDBM_FP64, 1, "p1x256");
    call(260, 260, PDBM_FP64, 3, "p2x484 p1x484");
    call(30, 5, PDBM_FP64, 3, "p2x4 p1x4");
    call(500, 1, PDBM_FP64, 25, "p24x7 p1x7");
    // ... and beyond marched, in blocks of two rows
    for (int precision : {PDBM_FP64, PDBM_FP32}) call(300, 300, precision, 1, "m1x750");
    call(300, 300, PDBM_FP64, 5, "p2x625 p2x625 m1x750");
    call(10, 9000, PDBM_FP32, 1, "m1x705");
    call(700, 150, PDBM_FP64, 1, "p1x767");
    // marched: blocks that fill rounds, of pairs and of single steps
    call(4000, 25, PDBM_FP32, 1, "m1x2000");
    call(330, 333, PDBM_FP64, 1, "m1x990");
    call(1100, 1024, PDBM_FP64, 3, "d2x1968 m1x1968");
    call(60000, 1, PDBM_FP64, 9, "c8x1250 c1x1250");
    // captured: an even number of launches where that of marching launches is
    call(64, 64, PDBM_FP64, 4, "p2x256 p2x256", true);
    call(300, 300, PDBM_FP64, 2, "p2x625", true);
    call(300, 300, PDBM_FP64, 3, "p2x625 m1x750", true);
    call(500, 1, PDBM_FP64, 16, "p8x7 p8x7", true);
    if (!fails) std::printf("launches ok\n");
    return fails ? 1 : 0;
}
