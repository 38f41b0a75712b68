// C ABI of the batched path: many independent systems (a block-diagonal
// matrix) with R right-hand sides each, solved by PP-GMRES in lockstep. Each
// system has its own polynomial (its own harmonic Ritz values), each
// (system, right-hand side) pair its own Krylov process, Hessenberg matrix
// and stopping test; every chain step and every Gram-Schmidt pass is one
// launch for the whole batch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/ppgmres.h"
#include "batched.h"
#include "common.h"
#include "host_core.h"
#include "kernels.h"
#include "poly.h"

using namespace ppg;

namespace {

constexpr double kBreakdownTolB = 1e-14;
constexpr double kInnerEtaB[3] = {0.0, 1e-5, 1e-2};
constexpr int kBlockRows = kBatchBlockRows;

struct BWork {
    int m = -1, R = 0;
    long ldv = 0;
    void *V = nullptr;
    void *buf = nullptr;  // P0 | P1 | T | D | ACC
    long vec = 0;         // bytes per vector
    void *P(int i) const { return (char *)buf + (size_t)i * vec; }
};

}  // namespace

struct pp_batch_s {
    // stream of graph-mode solves: the caller's stream may be the legacy
    // default stream, which cannot be captured (created on first use,
    // default priority, non-blocking)
    hipStream_t gstream = nullptr;
    hipEvent_t gevent = nullptr;
    int nsys = 0;
    long n = 0, nnz = 0;
    std::vector<long> row_off;
    // sliced-ELL of the batch
    int4 *slice = nullptr;
    int32_t *sptr = nullptr, *scol = nullptr, *sperm = nullptr;
    double *sval64 = nullptr;
    float *sval32 = nullptr;
    int nslices = 0;
    long npad = 0;
    // pattern-coded copy (format 1; see pp_batch_set_format)
    uint8_t *bpat = nullptr;
    // constant-coefficient box copy (format 2): per system its grid's line
    // length and its interior row's pattern; set only beside the pattern copy
    int32_t *bgx = nullptr, *bpint = nullptr;
    int has_box = 0;
    int32_t *poff = nullptr, *ptoff = nullptr, *sysoff = nullptr;
    double *ptab64 = nullptr;
    float *ptab32 = nullptr;
    int pnd = 0;
    int format = 0;
    // reduction blocks
    int4 *block = nullptr;
    int32_t *boff = nullptr;
    int nblocks = 0;
    // work
    BWork ws[3];
    int ldp = 0, ldh = 0;
    double *partial = nullptr, *npart = nullptr, *h1 = nullptr, *h2 = nullptr, *inv = nullptr;
    double *Hc = nullptr, *z = nullptr;      // pairs x ldh
    double *hpin = nullptr, *zpin = nullptr;  // pinned mirrors
    double *r64 = nullptr;                    // n*R (FP64)
    long r64_len = 0;
    int pairs_cap = 0;
    PStep *desc_spmv = nullptr, *desc_res = nullptr;  // nsys x 1 uniform programs

    int *act = nullptr;     // device: per-system active flags of the Arnoldi loop
    int *ones = nullptr;    // device: all systems active (the unmasked chain's flags)
    int *actpin = nullptr;  // pinned mirror
    int *kdev = nullptr;    // device: columns per pair of the last cycle
    int *kpin = nullptr;
    // device least squares of every pair (see BGivens), its per-cycle inputs
    // (beta | target | 1/beta per pair, run flags) and outputs (steps, last
    // shortcut residual), staged through pinned memory
    double *gR = nullptr, *gc = nullptr, *gs = nullptr, *gg = nullptr, *gfro = nullptr, *gsc = nullptr;
    double *gin = nullptr, *ginpin = nullptr, *gscpin = nullptr;
    int *grun = nullptr, *gsteps = nullptr, *grunpin = nullptr, *gstepspin = nullptr;
    int *gany = nullptr, *ganypin = nullptr;  // some pair still runs (device, pinned mirror)
    int gm = -1, gpairs = 0;
    // delayed Gram-Schmidt of the cycle (orth == 1): dot-pass partials and
    // their per-system sums (ldd = 2 (m + 1) R per row), every pair's
    // Hessenberg matrix (column c at dH + p*ldhp + c*(m+1)), pending and
    // next coefficients (m + 1 per pair) and {1/rho, g_j} per pair
    int orth = 1;
    int ldd = 0;
    double *dpart = nullptr, *ddot = nullptr, *dH = nullptr, *dpend = nullptr, *dg = nullptr, *dcoef = nullptr;
    void free_givens() {
        dev_free(dpart);
        dev_free(ddot);
        dev_free(dH);
        dev_free(dpend);
        dev_free(dg);
        dev_free(dcoef);
        ldd = 0;
        dev_free(gR);
        dev_free(gc);
        dev_free(gs);
        dev_free(gg);
        dev_free(gfro);
        dev_free(gsc);
        dev_free(gin);
        dev_free(grun);
        dev_free(gsteps);
        dev_free(gany);
        if (ganypin) (void)hipHostFree(ganypin);
        ganypin = nullptr;
        if (ginpin) (void)hipHostFree(ginpin);
        if (gscpin) (void)hipHostFree(gscpin);
        if (grunpin) (void)hipHostFree(grunpin);
        if (gstepspin) (void)hipHostFree(gstepspin);
        ginpin = gscpin = nullptr;
        grunpin = gstepspin = nullptr;
        gm = -1;
        gpairs = 0;
    }
    pp_status ensure_givens(int m, int R) {
        const int pairs = nsys * R;
        if (gm == m && gpairs == pairs) return PP_OK;
        free_givens();
        PP_TRY(dev_alloc(&gR, (size_t)pairs * (m + 1) * m));
        PP_TRY(dev_alloc(&gc, (size_t)pairs * m));
        PP_TRY(dev_alloc(&gs, (size_t)pairs * m));
        PP_TRY(dev_alloc(&gg, (size_t)pairs * (m + 1)));
        PP_TRY(dev_alloc(&gfro, (size_t)pairs));
        PP_TRY(dev_alloc(&gsc, (size_t)pairs));
        PP_TRY(dev_alloc(&gin, (size_t)3 * pairs));
        PP_TRY(dev_alloc(&grun, (size_t)pairs));
        PP_TRY(dev_alloc(&gsteps, (size_t)pairs));
        PP_TRY(dev_alloc(&gany, 1));
        ldd = 2 * (m + 1) * R;
        PP_TRY(dev_alloc(&dpart, (size_t)nblocks * ldd));
        PP_TRY(dev_alloc(&ddot, (size_t)nsys * ldd));
        PP_TRY(dev_alloc(&dH, (size_t)pairs * m * (m + 1)));
        PP_TRY(dev_alloc(&dpend, (size_t)pairs * (m + 1)));
        PP_TRY(dev_alloc(&dg, (size_t)pairs * (m + 1)));
        PP_TRY(dev_alloc(&dcoef, (size_t)pairs * 2));
        if (hipHostMalloc((void **)&ginpin, sizeof(double) * 3 * pairs, hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void **)&ganypin, sizeof(int), hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void **)&gscpin, sizeof(double) * pairs, hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void **)&grunpin, sizeof(int) * pairs, hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void **)&gstepspin, sizeof(int) * pairs, hipHostMallocDefault) != hipSuccess) {
            set_error("hipHostMalloc failed");
            return PP_ENOMEM;
        }
        gm = m;
        gpairs = pairs;
        return PP_OK;
    }
    BGivens givens(int R) const {
        BGivens G;
        G.Rm = gR;
        G.c = gc;
        G.s = gs;
        G.g = gg;
        G.fro2 = gfro;
        G.target = gin + gpairs;
        G.sc = gsc;
        G.run = grun;
        G.k = kdev;
        G.steps = gsteps;
        G.act = act;
        G.m = gm;
        G.R = R;
        G.nsys = nsys;
        return G;
    }
    // launch shape of the chain kernels per precision and right-hand-side
    // count, chosen by tune_bchain (format: 0 sliced-ELL, 1 pattern-coded)
    struct ChainCfg {
        int tuned = 0, format = 0, spw = 1, remap = 1;
        double us = 0.0;
    };
    ChainCfg cfg[3][5];
    // many steps per launch (box copy) per precision and right-hand-side
    // count: the tiles (grid_tiles, owned) and shape, steps 0: off
    BatchGrid grid[3][5];
    int4 *grid_tiles[3][5] = {};
    double grid_us[3][5] = {};
    void grid_off(int prec, int R) {
        dev_free(grid_tiles[prec][R]);
        grid[prec][R] = BatchGrid();
        grid_us[prec][R] = 0.0;
    }
    void grids_off() {
        for (int p = 0; p < 3; ++p)
            for (int r = 0; r < 5; ++r) grid_off(p, r);
    }
    std::vector<int32_t> h_bgx;  // line length of every system's grid (box copy)
    std::vector<std::pair<int, int>> grids() const {
        std::vector<std::pair<int, int>> g;
        for (int s = 0; s < nsys; ++s) g.emplace_back(h_bgx[s], (int)((row_off[s + 1] - row_off[s]) / h_bgx[s]));
        return g;
    }
    // The shape's tiles over every system, uploaded (both tile lists in one
    // allocation); off when a region leaves no tile.
    pp_status grid_on(int prec, int R, int ry, int waves, int steps, hipStream_t st) {
        grid_off(prec, R);
        const int aw = batch_grid_acc_waves(prec, R, ry, waves);
        const auto gs = grids();
        if (!batch_grid_fits(prec, R, ry, waves, steps, gs)) return PP_OK;
        std::vector<int4> t;
        size_t first = 0;
        for (int h : {ry * waves, ry * aw}) {
            first = t.size();
            for (int s = 0; s < nsys; ++s) {
                int tx, ty;
                batch_grid_tile(gs[s].first, gs[s].second, h, steps, &tx, &ty);
                for (int y = 0; y < gs[s].second; y += ty)
                    for (int x = 0; x < gs[s].first; x += tx) t.push_back(int4{s, x, y, 0});
            }
        }
        PP_TRY(dev_alloc(&grid_tiles[prec][R], t.size()));
        HIP_TRY(hipMemcpyAsync(grid_tiles[prec][R], t.data(), sizeof(int4) * t.size(), hipMemcpyHostToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        BatchGrid &g = grid[prec][R];
        g.tile = grid_tiles[prec][R];
        g.ntiles = (int)first;
        g.acc_tile = g.tile + first;
        g.acc_ntiles = (int)(t.size() - first);
        g.ry = ry;
        g.waves = waves;
        g.acc_waves = aw;
        g.steps = steps;
        return PP_OK;
    }
    bool format_forced = false;  // pp_batch_set_format: the tuner keeps the format
    bool format_ok(int f) const { return f == 0 || (f == 1 && pnd > 0) || (f == 2 && has_box && pnd > 0); }
    // use_box: the box copy whatever the format (the multi-step kernel's)
    BatchSell sell(int prec, bool masked = false, int R = 1, bool use_box = false) const {
        const ChainCfg &c = cfg[prec][R];
        const int fmt = use_box ? 2 : (c.tuned && !format_forced && format_ok(c.format)) ? c.format : format;
        BatchSell s;
        s.spw = c.tuned ? c.spw : 1;
        s.remap = c.tuned ? c.remap : 1;
        s.active = masked ? act : ones;
        s.slice = slice;
        s.sptr = sptr;
        s.scol = scol;
        s.sval64 = sval64;
        s.sval32 = sval32;
        s.nslices = nslices;
        const bool pat = (fmt == 1 || fmt == 2) && pnd > 0;
        const bool box = fmt == 2 && has_box && pnd > 0;
        s.bgx = box ? bgx : nullptr;
        s.bpint = box ? bpint : nullptr;
        s.bpat = pat ? bpat : nullptr;
        s.poff = pat ? poff : nullptr;
        s.ptoff = pat ? ptoff : nullptr;
        s.sysoff = pat ? sysoff : nullptr;
        s.ptab64 = pat ? ptab64 : nullptr;
        s.ptab32 = pat ? ptab32 : nullptr;
        s.pnd = pat ? pnd : 0;
        return s;
    }
    void drop_patterns() {
        dev_free(bgx);
        dev_free(bpint);
        has_box = 0;
        dev_free(bpat);
        dev_free(poff);
        dev_free(ptoff);
        dev_free(sysoff);
        dev_free(ptab64);
        dev_free(ptab32);
        pnd = 0;
        format = 0;
        grids_off();
    }
    BatchBlocks blocks(bool masked = false) const {
        BatchBlocks b;
        b.active = masked ? act : nullptr;
        b.block = block;
        b.boff = boff;
        b.nblocks = nblocks;
        b.nsys = nsys;
        return b;
    }
    void free_ws(BWork &w) {
        dev_free(w.V);
        dev_free(w.buf);
        w.m = -1;
        w.R = 0;
    }
    pp_status ensure(int prec, int m, int R) {
        BWork &w = ws[prec];
        if (w.m >= m && w.R == R && w.V) return PP_OK;
        free_ws(w);
        const size_t es = elem_size(prec);
        w.ldv = (n * R + 63) / 64 * 64;
        w.vec = (long)(w.ldv * es);
        char *p = nullptr;
        PP_TRY(dev_alloc(&p, (size_t)w.vec * (m + 1)));
        w.V = p;
        char *q = nullptr;
        PP_TRY(dev_alloc(&q, (size_t)w.vec * 5));
        w.buf = q;
        w.m = m;
        w.R = R;
        return PP_OK;
    }
    // reduction buffers for `cols` Krylov columns and R right-hand sides
    pp_status ensure_red(int cols, int R) {
        const int want_p = (cols + 2) * R;
        const int pairs = nsys * R;
        if (want_p <= ldp && cols + 2 <= ldh && pairs <= pairs_cap && (long)n * R <= r64_len) return PP_OK;
        dev_free(partial);
        dev_free(npart);
        dev_free(h1);
        dev_free(h2);
        dev_free(inv);
        dev_free(Hc);
        dev_free(z);
        dev_free(r64);
        dev_free(kdev);
        if (hpin) (void)hipHostFree(hpin);
        if (zpin) (void)hipHostFree(zpin);
        if (kpin) (void)hipHostFree(kpin);
        hpin = zpin = nullptr;
        kpin = nullptr;
        ldp = std::max(want_p, 64);
        ldh = std::max(cols + 2, 64);
        pairs_cap = pairs;
        r64_len = (long)n * R;
        PP_TRY(dev_alloc(&partial, (size_t)nblocks * ldp));
        PP_TRY(dev_alloc(&npart, (size_t)nblocks * R));
        PP_TRY(dev_alloc(&h1, (size_t)nsys * ldp));
        PP_TRY(dev_alloc(&h2, (size_t)nsys * ldp));
        PP_TRY(dev_alloc(&inv, (size_t)pairs));
        PP_TRY(dev_alloc(&Hc, (size_t)pairs * ldh));
        PP_TRY(dev_alloc(&z, (size_t)pairs * ldh));
        PP_TRY(dev_alloc(&r64, (size_t)n * R));
        PP_TRY(dev_alloc(&kdev, (size_t)pairs));
        if (hipHostMalloc((void **)&hpin, sizeof(double) * pairs * ldh, hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void **)&zpin, sizeof(double) * pairs * ldh, hipHostMallocDefault) != hipSuccess ||
            hipHostMalloc((void **)&kpin, sizeof(int) * pairs, hipHostMallocDefault) != hipSuccess) {
            set_error("hipHostMalloc failed");
            return PP_ENOMEM;
        }
        return PP_OK;
    }
    ~pp_batch_s() {
        if (gstream) {
            (void)hipStreamSynchronize(gstream);
            (void)hipStreamDestroy(gstream);
        }
        if (gevent) (void)hipEventDestroy(gevent);
        free_givens();
        for (auto &w : ws) free_ws(w);
        dev_free(slice);
        dev_free(sptr);
        dev_free(scol);
        dev_free(sperm);
        dev_free(sval64);
        dev_free(sval32);
        drop_patterns();
        dev_free(block);
        dev_free(boff);
        dev_free(partial);
        dev_free(npart);
        dev_free(h1);
        dev_free(h2);
        dev_free(inv);
        dev_free(Hc);
        dev_free(z);
        dev_free(r64);
        dev_free(desc_spmv);
        dev_free(desc_res);
        dev_free(act);
        dev_free(ones);
        grids_off();
        dev_free(kdev);
        if (actpin) (void)hipHostFree(actpin);
        if (kpin) (void)hipHostFree(kpin);
        if (hpin) (void)hipHostFree(hpin);
        if (zpin) (void)hipHostFree(zpin);
    }
};

namespace {

PStep pstep_of(const Step &s) {
    PStep p;
    std::memset(&p, 0, sizeof(p));
    p.spmv = s.spmv;
    p.in = s.in;
    p.aux = s.aux;
    p.out = s.out;
    p.acc = s.acc;
    p.acc_init = s.acc_init;
    p.fin = s.fin;
    p.a0 = s.a0;
    p.a1 = s.a1;
    p.a2 = s.a2;
    p.b0 = s.b0;
    p.b1 = s.b1;
    return p;
}

PStep skip_step() {
    PStep p;
    std::memset(&p, 0, sizeof(p));
    p.spmv = -1;
    p.in = 0;
    p.aux = p.out = p.acc = -1;
    return p;
}

pp_status upload(const std::vector<PStep> &h, PStep **dst, hipStream_t st) {
    PP_TRY(dev_alloc(dst, h.size()));
    HIP_TRY(hipMemcpyAsync(*dst, h.data(), sizeof(PStep) * h.size(), hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    return PP_OK;
}

// Per-system programs of one kind, padded to a common length K with skipped
// steps, and per precision their segments for the multi-step kernel (L
// launches; null: one launch per step).
struct BatchProg {
    PStep *steps = nullptr;
    int K = 0;
    BatchSeg *segs[3] = {nullptr, nullptr, nullptr};
    int L[3] = {0, 0, 0};
    bool acc = false;  // the programs have an accumulator
    ~BatchProg() {
        dev_free(steps);
        for (auto &p : segs) dev_free(p);
    }
};

const std::vector<Step> &prog_of(const pp_poly p, int kind) { return kind == PP_APPLY_P ? p->prog_p : p->prog_phi; }

pp_status upload_programs(pp_batch B, const pp_poly *polys, int kind, BatchProg &P, hipStream_t st) {
    int kmax = 0;
    for (int s = 0; s < B->nsys; ++s) kmax = std::max(kmax, (int)prog_of(polys[s], kind).size());
    std::vector<PStep> h((size_t)B->nsys * kmax, skip_step());
    for (int s = 0; s < B->nsys; ++s) {
        const auto &prog = prog_of(polys[s], kind);
        for (size_t k = 0; k < prog.size(); ++k) h[(size_t)s * kmax + k] = pstep_of(prog[k]);
    }
    P.K = kmax;
    P.acc = kind == PP_APPLY_P;
    return upload(h, &P.steps, st);
}

// The programs' segments for precision prec's multi-step launches, if it has
// them and every program is one chain. Each system cuts its own program; one
// with fewer segments than the longest sits out the last launches.
pp_status upload_segments(pp_batch B, const pp_poly *polys, int kind, int prec, int R, BatchProg &P, hipStream_t st) {
    const int smax = B->grid[prec][R].steps;
    if (smax == 0 || P.segs[prec]) return PP_OK;
    std::vector<std::vector<int>> lens(B->nsys);
    int L = 0;
    for (int s = 0; s < B->nsys; ++s) {
        const auto &prog = prog_of(polys[s], kind);
        if (!linear_program(prog) || (prog[0].acc != B_NONE) != P.acc) return PP_OK;
        lens[s] = split_program(prog, smax);
        L = std::max(L, (int)lens[s].size());
    }
    std::vector<BatchSeg> h((size_t)B->nsys * L);
    std::memset(h.data(), 0, sizeof(BatchSeg) * h.size());
    for (int s = 0; s < B->nsys; ++s) {
        const auto &prog = prog_of(polys[s], kind);
        int i = 0, from = B_IN, to = B_P0;
        for (size_t l = 0; l < lens[s].size(); ++l) {
            const bool last = l + 1 == lens[s].size();
            BatchSeg &g = h[(size_t)s * L + l];
            g.first = i;
            g.count = lens[s][l];
            g.in = from;
            g.out = last ? prog.back().out : to;
            g.fin = last ? prog.back().fin : 0;
            g.acc = prog[i].acc;
            g.acc_init = prog[i].acc_init;
            from = to;
            to = to == B_P0 ? B_P1 : B_P0;
            i += g.count;
        }
    }
    PP_TRY(dev_alloc(&P.segs[prec], h.size()));
    HIP_TRY(hipMemcpyAsync(P.segs[prec], h.data(), sizeof(BatchSeg) * h.size(), hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    P.L[prec] = L;
    return PP_OK;
}

pp_status run_bprog(pp_batch B, int prec, int R, const BatchProg &P, const void *in, void *out, const BWork &w,
                    hipStream_t st, bool masked = false) {
    void *bufs[5] = {(void *)in, out, w.P(0), w.P(1), w.P(2)};
    if (P.segs[prec]) {
        const BatchSell X = B->sell(prec, masked, R, true);
        for (int l = 0; l < P.L[prec]; ++l)
            HIP_TRY(launch_bgrid(X, B->grid[prec][R], P.acc, prec, R, P.steps, P.K, P.segs[prec], P.L[prec], l, bufs, st));
        return PP_OK;
    }
    const BatchSell S = B->sell(prec, masked, R);
    for (int k = 0; k < P.K; ++k) HIP_TRY(launch_bchain(S, prec, R, P.steps, P.K, k, bufs, st));
    return PP_OK;
}

// The batched autotuner: one sparse product over the whole batch (every
// system active) is timed for each storage format the batch has (unless the
// caller fixed it), slices per wave (1 or 2, pattern-coded format) and
// workgroup order (XCD-aware or not), on the batch's own matrix, precision
// and right-hand-side count; the fastest is kept for (prec, R).
pp_status tune_bgrid(pp_batch B, int prec, int R, double single, hipEvent_t e0, hipEvent_t e1, hipStream_t st);

pp_status tune_bchain(pp_batch B, int prec, int R, hipStream_t st) {
    PP_TRY(B->ensure(prec, std::max(B->ws[prec].m, 1), R));
    const BWork &w = B->ws[prec];
    HIP_TRY(hipMemsetAsync(w.P(0), 0, (size_t)w.vec, st));
    void *bufs[5] = {w.P(0), w.P(1), w.P(2), w.P(3), w.P(4)};
    hipEvent_t e0, e1;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    struct EvGuard {
        hipEvent_t a, b;
        ~EvGuard() {
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
        }
    } guard{e0, e1};
    pp_batch_s::ChainCfg &c = B->cfg[prec][R];
    pp_batch_s::ChainCfg best;
    best.us = 1e30;
    const int reps = 5;
    for (int fmt = 2; fmt >= 0; --fmt) {
        if (!B->format_ok(fmt)) continue;
        if (B->format_forced && fmt != B->format) continue;
        for (int spw = 1; spw <= (fmt >= 1 ? 2 : 1); ++spw)
            for (int remap = 0; remap <= 1; ++remap) {
                c.tuned = 1;
                c.format = fmt;
                c.spw = spw;
                c.remap = remap;
                const BatchSell S = B->sell(prec, false, R);
                double t = 1e30;
                for (int round = 0; round < 2; ++round) {
                    for (int i = 0; i < 2; ++i) HIP_TRY(launch_bchain(S, prec, R, B->desc_spmv, 1, 0, bufs, st));
                    HIP_TRY(hipEventRecord(e0, st));
                    for (int i = 0; i < reps; ++i) HIP_TRY(launch_bchain(S, prec, R, B->desc_spmv, 1, 0, bufs, st));
                    HIP_TRY(hipEventRecord(e1, st));
                    HIP_TRY(hipEventSynchronize(e1));
                    float ms = 0.f;
                    HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
                    t = std::min(t, 1e3 * ms / reps);
                }
                if (t < best.us) {
                    best = c;
                    best.us = t;
                }
            }
    }
    c = best;
    c.tuned = 1;
    const pp_status g = tune_bgrid(B, prec, R, best.us, e0, e1, st);
    if (g != PP_OK) c.tuned = 0;
    return g;
}

// Times the multi-step kernel's shapes over the whole batch (when it has the
// box copy and the caller forced no format) and turns on the one with the
// lowest time per step if that beats `single`, the best single-step launch. The
// shapes timed are the four most promising (batch_grid_shapes).
pp_status tune_bgrid(pp_batch B, int prec, int R, double single, hipEvent_t e0, hipEvent_t e1, hipStream_t st) {
    B->grid_off(prec, R);
    if (B->format_forced || !B->format_ok(2)) return PP_OK;
    const std::vector<BatchGridShape> all = batch_grid_shapes(prec, R, B->grids());
    const BWork &w = B->ws[prec];
    // a program of the most steps: real roots, no accumulator
    BatchProg P;
    std::vector<PStep> h((size_t)B->nsys * kGrid2MaxSteps, pstep_of(Step{1, B_P0, B_NONE, B_P1, B_NONE, 0, 0, 1.0, 0.0, 0.0, 0.0, 0.0}));
    PP_TRY(upload(h, &P.steps, st));
    PP_TRY(dev_alloc(&P.segs[prec], B->nsys));
    void *bufs[5] = {w.P(0), w.P(1), w.P(2), w.P(3), w.P(4)};
    BatchGridShape best{single, 0, 0, 0};
    for (size_t k = 0; k < all.size() && k < 4; ++k) {
        const BatchGridShape &c = all[k];
        PP_TRY(B->grid_on(prec, R, c.ry, c.waves, c.steps, st));
        if (B->grid[prec][R].steps == 0) continue;
        std::vector<BatchSeg> sg(B->nsys, BatchSeg{0, c.steps, B_IN, B_OUT, 0, -1, 0, 0});
        HIP_TRY(hipMemcpyAsync(P.segs[prec], sg.data(), sizeof(BatchSeg) * sg.size(), hipMemcpyHostToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        const BatchSell S = B->sell(prec, false, R, true);
        double us = 1e30;
        for (int round = 0; round < 2; ++round) {
            HIP_TRY(launch_bgrid(S, B->grid[prec][R], false, prec, R, P.steps, kGrid2MaxSteps, P.segs[prec], 1, 0, bufs, st));
            HIP_TRY(hipEventRecord(e0, st));
            for (int i = 0; i < 3; ++i)
                HIP_TRY(launch_bgrid(S, B->grid[prec][R], false, prec, R, P.steps, kGrid2MaxSteps, P.segs[prec], 1, 0, bufs, st));
            HIP_TRY(hipEventRecord(e1, st));
            HIP_TRY(hipEventSynchronize(e1));
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
            us = std::min(us, 1e3 * ms / 3);
        }
        if (us / c.steps < best.t) best = BatchGridShape{us / c.steps, c.ry, c.waves, c.steps};
    }
    B->grid_off(prec, R);
    if (best.steps == 0) return PP_OK;
    PP_TRY(B->grid_on(prec, R, best.ry, best.waves, best.steps, st));
    B->grid_us[prec][R] = best.t * best.steps;
    return PP_OK;
}

void *bcol(const BWork &w, int prec, int j) { return (char *)w.V + (size_t)j * w.ldv * elem_size(prec); }

// CGS2 of column j+1 against columns 0..j for every pair; H column base
// Hbase (pair stride pstride): H[0..j] and H[j+1] = norm; w normalised.
pp_status bcgs2(pp_batch B, int prec, int R, const BWork &w, int j, double *Hbase, long pstride, hipStream_t st,
                bool masked = false) {
    const BatchBlocks bl = B->blocks(masked);
    const int ncols = j + 1;
    void *wv = bcol(w, prec, j + 1);
    HIP_TRY(launch_bdots(bl, prec, R, w.V, w.ldv, ncols, wv, B->partial, B->ldp, st));
    HIP_TRY(launch_bred(bl, R, B->partial, B->ldp, ncols * R, B->h1, B->ldp, Hbase, pstride, 1, st));
    if (ncols <= bupdate_dots_max_cols(prec)) {
        // w -= V h1 with h2 = V^T w and ||w||^2 from the same read of V; then
        // H += h2, the norm from ||w||^2 - ||h2||^2, and w = (w - V h2) / norm
        // in one more read
        HIP_TRY(launch_bupdate_dots(bl, prec, R, w.V, w.ldv, ncols, B->h1, B->ldp, wv, B->partial, B->ldp, st));
        HIP_TRY(launch_bred(bl, R, B->partial, B->ldp, ncols * R + R, B->h2, B->ldp, nullptr, 0, 0, st));
        HIP_TRY(launch_bfinish(bl, R, ncols, B->h2, B->ldp, Hbase, pstride, B->inv, st));
        HIP_TRY(launch_bupdate(bl, prec, R, w.V, w.ldv, ncols, B->h2, B->ldp, wv, nullptr, B->inv, st));
        return PP_OK;
    }
    HIP_TRY(launch_bupdate(bl, prec, R, w.V, w.ldv, ncols, B->h1, B->ldp, wv, nullptr, nullptr, st));
    HIP_TRY(launch_bdots(bl, prec, R, w.V, w.ldv, ncols, wv, B->partial, B->ldp, st));
    HIP_TRY(launch_bred(bl, R, B->partial, B->ldp, ncols * R, B->h2, B->ldp, Hbase, pstride, 2, st));
    HIP_TRY(launch_bupdate(bl, prec, R, w.V, w.ldv, ncols, B->h2, B->ldp, wv, B->npart, nullptr, st));
    HIP_TRY(launch_bnorm(bl, R, B->npart, Hbase + ncols, pstride, B->inv, st));
    HIP_TRY(launch_bscale(bl, prec, prec, R, wv, B->inv, wv, st));
    return PP_OK;
}

// Step j of the delayed Gram-Schmidt for every pair (masked): the dot pass
// of the pending vector u (w.P(3)) and w = phi(A) u (column j+1) against
// columns 0..j-1, the per-system sums, the coefficient step (Hessenberg
// column j-1 complete) and, unless final, the update pass (column j = v_j,
// u = the next pending vector). final: the cycle's last call (j = m), which
// only completes column m-1.
pp_status bdcgs(pp_batch B, int prec, int R, const BWork &w, int j, bool final, hipStream_t st) {
    const BatchBlocks bl = B->blocks(true);
    const int m = B->gm, ldc = m + 1;
    void *u = w.P(3);
    const void *wv = final ? u : bcol(w, prec, j + 1);
    HIP_TRY(launch_bdots2(bl, prec, R, w.V, w.ldv, j, u, wv, B->dpart, B->ldd, st));
    HIP_TRY(launch_bred(bl, R, B->dpart, B->ldd, 2 * (j + 1) * R, B->ddot, B->ldd, nullptr, 0, 0, st));
    HIP_TRY(launch_bdcgs_step(bl, R, j, B->ddot, B->ldd, B->dH, (long)m * ldc, ldc, B->dpend, B->dg, B->dcoef,
                              final ? 1 : 0, st));
    if (!final)
        HIP_TRY(launch_bupdate2(bl, prec, R, w.V, w.ldv, j, B->ddot, B->ldd, B->dg, ldc, B->dcoef, u,
                                bcol(w, prec, j + 1), bcol(w, prec, j), st));
    return PP_OK;
}

// ||v_p|| for every pair of an FP64 vector (synchronises; result in out[p])
pp_status bnorms(pp_batch B, int R, const double *v, std::vector<double> &out, hipStream_t st) {
    const BatchBlocks bl = B->blocks();
    HIP_TRY(launch_bdots(bl, 0, R, v, 0, 1, v, B->partial, B->ldp, st));
    HIP_TRY(launch_bred(bl, R, B->partial, B->ldp, R, B->h1, B->ldp, nullptr, 0, 0, st));
    // h1[s*ldp + r] -> host
    HIP_TRY(hipMemcpy2DAsync(B->hpin, sizeof(double) * R, B->h1, sizeof(double) * B->ldp, sizeof(double) * R, B->nsys,
                             hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    out.resize((size_t)B->nsys * R);
    for (size_t p = 0; p < out.size(); ++p) out[p] = std::sqrt(B->hpin[p]);
    return PP_OK;
}

}  // namespace

namespace {

// The pattern-coded copy (format 1): every system's entries on the same
// number nd of diagonals (its own offsets), at most 256 distinct rows per
// system (a row is the tuple of its nd values, 0 where it has no entry).
// Leaves the batch without the copy (PP_OK) when it does not qualify.
pp_status build_batch_patterns(pp_batch B, const std::vector<int32_t> &rp, const std::vector<int32_t> &ci,
                               const double *val, hipStream_t st) {
    const int nsys = B->nsys;
    const long n = B->n;
    if (B->nnz == 0) return PP_OK;
    int nd = -1;
    std::vector<int32_t> offs;
    for (int s = 0; s < nsys; ++s) {
        std::vector<int32_t> o;
        for (long r = B->row_off[s]; r < B->row_off[s + 1]; ++r)
            for (int e = rp[r]; e < rp[r + 1]; ++e) {
                const int32_t d = ci[e] - (int32_t)r;
                if (std::find(o.begin(), o.end(), d) == o.end()) {
                    o.push_back(d);
                    if ((int)o.size() > kMaxDiag) return PP_OK;
                }
            }
        std::sort(o.begin(), o.end());
        if (nd < 0) nd = (int)o.size();
        if ((int)o.size() != nd) return PP_OK;
        offs.insert(offs.end(), o.begin(), o.end());
    }
    if (!(nd == 3 || nd == 5 || nd == 7 || nd == 9 || nd == 13 || nd == 19 || nd == 27)) return PP_OK;
    std::vector<double> hv(B->nnz);
    if (hipMemcpyAsync(hv.data(), val, sizeof(double) * B->nnz, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess) {
        set_error("pp_batch_create: cannot read the values");
        return PP_EDEVICE;
    }
    std::vector<uint8_t> pid((size_t)n, 0);
    std::vector<double> tab;
    std::vector<int32_t> toff(nsys), so(nsys + 1);
    std::vector<double> tup(nd);
    std::vector<char> seen(nd);
    for (int s = 0; s < nsys; ++s) {
        toff[s] = (int32_t)tab.size();
        so[s] = (int32_t)B->row_off[s];
        const int32_t *o = offs.data() + (size_t)s * nd;
        std::unordered_map<std::string, int> id_of;
        std::string prev;
        int prev_id = -1;
        for (long r = B->row_off[s]; r < B->row_off[s + 1]; ++r) {
            std::fill(tup.begin(), tup.end(), 0.0);
            std::fill(seen.begin(), seen.end(), 0);
            for (int e = rp[r]; e < rp[r + 1]; ++e) {
                const int d = (int)(std::lower_bound(o, o + nd, ci[e] - (int32_t)r) - o);
                if (seen[d]) return PP_OK;  // two entries of one column
                seen[d] = 1;
                tup[d] = hv[e];
            }
            std::string key(reinterpret_cast<const char *>(tup.data()), sizeof(double) * nd);
            int id = prev_id;
            if (prev_id < 0 || key != prev) {
                auto it = id_of.find(key);
                if (it == id_of.end()) {
                    if (id_of.size() >= 256) return PP_OK;
                    id = (int)id_of.size();
                    id_of.emplace(key, id);
                    tab.insert(tab.end(), tup.begin(), tup.end());
                } else {
                    id = it->second;
                }
                prev = std::move(key);
                prev_id = id;
            }
            pid[r] = (uint8_t)id;
        }
        if (tab.size() >= (size_t)1 << 31) return PP_OK;
    }
    so[nsys] = (int32_t)n;
    // constant-coefficient box stencils (5-point): system s's offsets are
    // -g, -1, 0, 1, g on a g-wide grid of at least 3 x 3 points, and every
    // row's tuple is its interior row's with the entries outside the grid
    // zero
    std::vector<int32_t> bg(nsys, 0), bp(nsys, 0);
    bool box = nd == 5;
    for (int s = 0; s < nsys && box; ++s) {
        const int32_t *o = offs.data() + (size_t)s * nd;
        const long base = B->row_off[s], ns = B->row_off[s + 1] - base;
        const long g = o[4];
        if (!(o[0] == -g && o[1] == -1 && o[2] == 0 && o[3] == 1 && g >= 3 && ns % g == 0 && ns / g >= 3)) {
            box = false;
            break;
        }
        const long gy = ns / g;
        const int pint = pid[(size_t)(base + g / 2 + g * (gy / 2))];
        const double *ci0 = tab.data() + (size_t)toff[s] + (size_t)pint * nd;
        for (long r = 0; r < ns && box; ++r) {
            const long x = r % g, y = r / g;
            const bool in[5] = {y > 0, x > 0, true, x + 1 < g, y + 1 < gy};
            const double *cr = tab.data() + (size_t)toff[s] + (size_t)pid[(size_t)(base + r)] * nd;
            for (int d = 0; d < nd; ++d)
                if (cr[d] != (in[d] ? ci0[d] : 0.0)) box = false;
        }
        bg[s] = (int32_t)g;
        bp[s] = pint;
    }
    std::vector<float> tab32(tab.size());
    for (size_t q = 0; q < tab.size(); ++q) tab32[q] = (float)tab[q];
    PP_TRY(dev_alloc(&B->bpat, pid.size()));
    PP_TRY(dev_alloc(&B->poff, offs.size()));
    PP_TRY(dev_alloc(&B->ptoff, toff.size()));
    PP_TRY(dev_alloc(&B->sysoff, so.size()));
    PP_TRY(dev_alloc(&B->ptab64, tab.size()));
    PP_TRY(dev_alloc(&B->ptab32, tab.size()));
    if (hipMemcpyAsync(B->bpat, pid.data(), pid.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->poff, offs.data(), sizeof(int32_t) * offs.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->ptoff, toff.data(), sizeof(int32_t) * toff.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->sysoff, so.data(), sizeof(int32_t) * so.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->ptab64, tab.data(), sizeof(double) * tab.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->ptab32, tab32.data(), sizeof(float) * tab.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess) {
        set_error("pp_batch_create: pattern-coded upload failed");
        return PP_EDEVICE;
    }
    B->pnd = nd;
    B->format = 1;
    if (box) {
        PP_TRY(dev_alloc(&B->bgx, bg.size()));
        PP_TRY(dev_alloc(&B->bpint, bp.size()));
        if (hipMemcpyAsync(B->bgx, bg.data(), sizeof(int32_t) * bg.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
            hipMemcpyAsync(B->bpint, bp.data(), sizeof(int32_t) * bp.size(), hipMemcpyHostToDevice, st) !=
                hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            set_error("pp_batch_create: box-stencil upload failed");
            return PP_EDEVICE;
        }
        B->has_box = 1;
        B->h_bgx = bg;
    }
    return PP_OK;
}

}  // namespace

extern "C" {

pp_status pp_batch_create(int nsys, const int64_t *row_off, int64_t nnz, const int32_t *rowptr, const int32_t *colind,
                          const double *val, void *stream, pp_batch *out) {
    if (nsys <= 0 || !row_off || !rowptr || !out || nnz < 0 || nnz >= (1LL << 31) || (nnz > 0 && (!colind || !val))) {
        set_error("pp_batch_create: bad argument");
        return PP_EINVAL;
    }
    const int64_t n = row_off[nsys];
    if (row_off[0] != 0 || n <= 0 || n >= (1LL << 31)) {
        set_error("pp_batch_create: row offsets must start at 0 and end below 2^31");
        return PP_EINVAL;
    }
    for (int s = 0; s < nsys; ++s)
        if (row_off[s + 1] <= row_off[s]) {
            set_error("pp_batch_create: every system needs at least one row");
            return PP_EINVAL;
        }
    hipStream_t st = S(stream);
    auto *B = new (std::nothrow) pp_batch_s();
    if (!B) return PP_ENOMEM;
    auto fail = [&](pp_status s) {
        delete B;
        return s;
    };
    B->nsys = nsys;
    B->n = n;
    B->nnz = nnz;
    B->row_off.assign(row_off, row_off + nsys + 1);
    std::vector<int32_t> rp(n + 1), ci(nnz);
    if (hipMemcpyAsync(rp.data(), rowptr, sizeof(int32_t) * (n + 1), hipMemcpyDeviceToHost, st) != hipSuccess ||
        (nnz && hipMemcpyAsync(ci.data(), colind, sizeof(int32_t) * nnz, hipMemcpyDeviceToHost, st) != hipSuccess) ||
        hipStreamSynchronize(st) != hipSuccess) {
        set_error("pp_batch_create: cannot read the pattern");
        return fail(PP_EDEVICE);
    }
    if (rp[0] != 0 || rp[n] != nnz) {
        set_error("pp_batch_create: rowptr[0] must be 0 and rowptr[n] must be nnz");
        return fail(PP_EINVAL);
    }
    // block-diagonal check: the columns of a row stay inside its system
    for (int s = 0; s < nsys; ++s)
        for (long r = row_off[s]; r < row_off[s + 1]; ++r) {
            if (rp[r + 1] < rp[r]) {
                set_error("pp_batch_create: rowptr not non-decreasing");
                return fail(PP_EINVAL);
            }
            for (int e = rp[r]; e < rp[r + 1]; ++e)
                if (ci[e] < row_off[s] || ci[e] >= row_off[s + 1]) {
                    set_error("pp_batch_create: entry outside its system's diagonal block");
                    return fail(PP_EINVAL);
                }
        }
    // sliced-ELL: 64-row slices inside each system
    std::vector<int4> sl;
    std::vector<int32_t> sp(1, 0);
    long tot = 0;
    for (int s = 0; s < nsys; ++s)
        for (long r0 = row_off[s]; r0 < row_off[s + 1]; r0 += 64) {
            const int nr = (int)std::min<long>(64, row_off[s + 1] - r0);
            int width = 0;
            for (int j = 0; j < nr; ++j) width = std::max(width, rp[r0 + j + 1] - rp[r0 + j]);
            sl.push_back(make_int4((int)r0, nr, s, 0));
            tot += 64L * width;
            if (tot >= (1L << 31)) {
                set_error("pp_batch_create: padded batch too large");
                return fail(PP_EINVAL);
            }
            sp.push_back((int32_t)tot);
        }
    std::vector<int32_t> scol(tot), sperm(tot, -1);
    for (size_t k = 0; k < sl.size(); ++k) {
        const int4 q = sl[k];
        const int width = (sp[k + 1] - sp[k]) / 64;
        for (int j = 0; j < 64; ++j) {
            const long r = (long)q.x + j;
            const int len = j < q.y ? rp[r + 1] - rp[r] : 0;
            for (int c = 0; c < width; ++c) {
                const long o = sp[k] + (long)c * 64 + j;
                if (c < len) {
                    scol[o] = ci[rp[r] + c];
                    sperm[o] = rp[r] + c;
                } else {
                    scol[o] = j < q.y ? (int32_t)r : q.x;  // padding: a valid row of the slice, value 0
                }
            }
        }
    }
    // reduction blocks
    std::vector<int4> bl;
    std::vector<int32_t> bo(1, 0);
    for (int s = 0; s < nsys; ++s) {
        for (long r0 = row_off[s]; r0 < row_off[s + 1]; r0 += kBlockRows)
            bl.push_back(make_int4((int)r0, (int)std::min<long>(kBlockRows, row_off[s + 1] - r0), s, 0));
        bo.push_back((int32_t)bl.size());
    }
    B->nslices = (int)sl.size();
    B->npad = tot;
    B->nblocks = (int)bl.size();
    pp_status s;
    if ((s = dev_alloc(&B->slice, sl.size())) != PP_OK || (s = dev_alloc(&B->sptr, sp.size())) != PP_OK ||
        (s = dev_alloc(&B->scol, (size_t)std::max<long>(tot, 1))) != PP_OK ||
        (s = dev_alloc(&B->sperm, (size_t)std::max<long>(tot, 1))) != PP_OK ||
        (s = dev_alloc(&B->sval64, (size_t)std::max<long>(tot, 1))) != PP_OK ||
        (s = dev_alloc(&B->sval32, (size_t)std::max<long>(tot, 1))) != PP_OK ||
        (s = dev_alloc(&B->block, bl.size())) != PP_OK || (s = dev_alloc(&B->boff, bo.size())) != PP_OK)
        return fail(s);
    if (hipMemcpyAsync(B->slice, sl.data(), sizeof(int4) * sl.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->sptr, sp.data(), sizeof(int32_t) * sp.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        (tot && hipMemcpyAsync(B->scol, scol.data(), sizeof(int32_t) * tot, hipMemcpyHostToDevice, st) != hipSuccess) ||
        (tot && hipMemcpyAsync(B->sperm, sperm.data(), sizeof(int32_t) * tot, hipMemcpyHostToDevice, st) != hipSuccess) ||
        hipMemcpyAsync(B->block, bl.data(), sizeof(int4) * bl.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemcpyAsync(B->boff, bo.data(), sizeof(int32_t) * bo.size(), hipMemcpyHostToDevice, st) != hipSuccess ||
        launch_sell_values(tot, B->sperm, val, B->sval64, B->sval32, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess) {
        set_error("pp_batch_create: device upload failed");
        return fail(PP_EDEVICE);
    }
    // uniform programs: one plain sparse product, and the residual b - A x
    std::vector<PStep> d1(nsys), dr(nsys);
    for (int q = 0; q < nsys; ++q) {
        std::memset(&d1[q], 0, sizeof(PStep));
        d1[q].spmv = 1;
        d1[q].in = B_IN;
        d1[q].out = B_OUT;
        d1[q].aux = d1[q].acc = -1;
        d1[q].a0 = 1.0;
        dr[q] = d1[q];
        dr[q].aux = B_P0;  // b
        dr[q].a0 = -1.0;
        dr[q].a2 = 1.0;
    }
    if ((s = upload(d1, &B->desc_spmv, st)) != PP_OK || (s = upload(dr, &B->desc_res, st)) != PP_OK) return fail(s);
    if ((s = dev_alloc(&B->act, (size_t)nsys)) != PP_OK) return fail(s);
    if ((s = dev_alloc(&B->ones, (size_t)nsys)) != PP_OK) return fail(s);
    {
        const std::vector<int> h1(nsys, 1);
        if (hipMemcpy(B->ones, h1.data(), sizeof(int) * nsys, hipMemcpyHostToDevice) != hipSuccess) {
            set_error("hipMemcpy failed");
            return fail(PP_EDEVICE);
        }
    }
    if ((s = build_batch_patterns(B, rp, ci, val, st)) != PP_OK) return fail(s);
    if (hipHostMalloc((void **)&B->actpin, sizeof(int) * nsys, hipHostMallocDefault) != hipSuccess) {
        B->actpin = nullptr;
        set_error("hipHostMalloc failed");
        return fail(PP_ENOMEM);
    }
    *out = B;
    return PP_OK;
}

void pp_batch_destroy(pp_batch B) { delete B; }

pp_status pp_batch_set_values(pp_batch B, const double *val, void *stream) {
    if (!B || (!val && B->nnz > 0)) {
        set_error("pp_batch_set_values: bad argument");
        return PP_EINVAL;
    }
    if (B->bpat) {
        // the patterns describe the old values
        (void)hipStreamSynchronize(S(stream));
        B->drop_patterns();
        B->format_forced = false;
    }
    for (auto &row : B->cfg)
        for (auto &c : row) c.tuned = 0;
    HIP_TRY(launch_sell_values(B->npad, B->sperm, val, B->sval64, B->sval32, S(stream)));
    return PP_OK;
}

pp_status pp_batch_set_format(pp_batch B, int format) {
    if (!B || format < 0 || format > 2) {
        set_error("pp_batch_set_format: bad argument");
        return PP_EINVAL;
    }
    if (format == 1 && !B->bpat) {
        set_error("pp_batch_set_format: no pattern-coded copy (the systems' diagonals or row patterns do not "
                  "qualify, or the values changed)");
        return PP_EINVAL;
    }
    if (format == 2 && !B->format_ok(2)) {
        set_error("pp_batch_set_format: no box-stencil copy (not every system is a constant-coefficient 5-point "
                  "stencil, or the values changed)");
        return PP_EINVAL;
    }
    B->format = format;
    B->format_forced = true;
    B->grids_off();
    for (auto &row : B->cfg)
        for (auto &c : row) c.tuned = 0;
    return PP_OK;
}

pp_status pp_batch_set_orth(pp_batch B, int delayed) {
    if (!B || (delayed != 0 && delayed != 1)) {
        set_error("pp_batch_set_orth: bad argument");
        return PP_EINVAL;
    }
    B->orth = delayed;
    return PP_OK;
}

pp_status pp_batch_orth(pp_batch B, int *delayed) {
    if (!B || !delayed) {
        set_error("pp_batch_orth: bad argument");
        return PP_EINVAL;
    }
    *delayed = B->orth;
    return PP_OK;
}

pp_status pp_batch_tune(pp_batch B, int prec, int nrhs, void *stream) {
    if (!B || prec < 0 || prec > 2 || !(nrhs == 1 || nrhs == 2 || nrhs == 4)) {
        set_error("pp_batch_tune: bad argument");
        return PP_EINVAL;
    }
    PP_TRY(tune_bchain(B, prec, nrhs, S(stream)));
    return PP_OK;
}

pp_status pp_batch_set_chain_config(pp_batch B, int prec, int nrhs, int format, int spw, int remap) {
    if (!B || prec < 0 || prec > 2 || !(nrhs == 1 || nrhs == 2 || nrhs == 4) || format < 0 || format > 2 ||
        spw < 1 || spw > 2 || remap < 0 || remap > 1 || (format == 0 && spw != 1)) {
        set_error("pp_batch_set_chain_config: bad argument (spw 2 only with the pattern-coded or box formats)");
        return PP_EINVAL;
    }
    if (format == 1 && !B->bpat) {
        set_error("pp_batch_set_chain_config: no pattern-coded copy");
        return PP_EINVAL;
    }
    if (format == 2 && !B->format_ok(2)) {
        set_error("pp_batch_set_chain_config: no box-stencil copy");
        return PP_EINVAL;
    }
    pp_batch_s::ChainCfg &c = B->cfg[prec][nrhs];
    c.tuned = 1;
    c.format = format;
    c.spw = spw;
    c.remap = remap;
    c.us = 0.0;
    B->format_forced = false;
    B->grid_off(prec, nrhs);
    return PP_OK;
}

pp_status pp_batch_set_grid(pp_batch B, int prec, int nrhs, int ry, int waves, int steps) {
    if (!B || prec < 0 || prec > 2 || !(nrhs == 1 || nrhs == 2 || nrhs == 4) || steps < 0) {
        set_error("pp_batch_set_grid: bad argument");
        return PP_EINVAL;
    }
    if (steps == 0) {
        B->grid_off(prec, nrhs);
        return PP_OK;
    }
    if (!B->format_ok(2) || B->format_forced || !B->cfg[prec][nrhs].tuned ||
        !batch_grid_ok(prec, nrhs, ry, waves, steps)) {
        set_error("pp_batch_set_grid: needs a box copy, no forced format, a tuned or set chain configuration and a "
                  "built shape, FP64 or FP32 vectors");
        return PP_EINVAL;
    }
    PP_TRY(B->grid_on(prec, nrhs, ry, waves, steps, 0));
    if (B->grid[prec][nrhs].steps == 0) {
        set_error("pp_batch_set_grid: the region leaves no tile");
        return PP_EINVAL;
    }
    return PP_OK;
}

pp_status pp_batch_grid(pp_batch B, int prec, int nrhs, int *shape, double *us) {
    if (!B || prec < 0 || prec > 2 || !(nrhs == 1 || nrhs == 2 || nrhs == 4) || !shape) {
        set_error("pp_batch_grid: bad argument");
        return PP_EINVAL;
    }
    const BatchGrid &g = B->grid[prec][nrhs];
    shape[0] = g.ry;
    shape[1] = g.waves;
    shape[2] = g.steps;
    if (us) *us = B->grid_us[prec][nrhs];
    return PP_OK;
}

pp_status pp_batch_chain_config(pp_batch B, int prec, int nrhs, int *format, int *spw, int *remap, double *us) {
    if (!B || prec < 0 || prec > 2 || !(nrhs == 1 || nrhs == 2 || nrhs == 4) || !format) {
        set_error("pp_batch_chain_config: bad argument");
        return PP_EINVAL;
    }
    const pp_batch_s::ChainCfg &c = B->cfg[prec][nrhs];
    const BatchSell S = B->sell(prec, false, nrhs);
    *format = S.bgx ? 2 : (S.bpat ? 1 : 0);
    if (spw) *spw = S.spw;
    if (remap) *remap = S.remap;
    if (us) *us = c.tuned ? c.us : 0.0;
    return PP_OK;
}

pp_status pp_batch_format(pp_batch B, int *format) {
    if (!B || !format) {
        set_error("pp_batch_format: bad argument");
        return PP_EINVAL;
    }
    *format = B->format;
    return PP_OK;
}

pp_status pp_batch_setup(pp_batch B, const double *v0, int d, int add_roots, void *stream, pp_poly *polys,
                         pp_setup_info *infos) {
    if (!B || !v0 || !polys || d < 1 || d > 4096) {
        set_error("pp_batch_setup: bad argument");
        return PP_EINVAL;
    }
    for (int s = 0; s < B->nsys; ++s)
        if (B->row_off[s + 1] - B->row_off[s] < d) {
            set_error("pp_batch_setup: degree above a system's size");
            return PP_EINVAL;
        }
    hipStream_t st = S(stream);
    const double t0 = now_s();
    const int R = 1, prec = 0;
    PP_TRY(B->ensure(prec, d, R));
    PP_TRY(B->ensure_red(d + 1, R));
    const BWork &w = B->ws[prec];
    const BatchBlocks bl = B->blocks();
    // V0 = v0 / ||v0|| per system
    void *v0c = bcol(w, prec, 0);
    HIP_TRY(hipMemcpyAsync(v0c, v0, sizeof(double) * B->n, hipMemcpyDeviceToDevice, st));
    HIP_TRY(launch_bupdate(bl, prec, R, w.V, w.ldv, 0, B->h1, B->ldp, v0c, B->npart, nullptr, st));
    HIP_TRY(launch_bnorm(bl, R, B->npart, nullptr, 0, B->inv, st));
    HIP_TRY(launch_bscale(bl, prec, prec, R, v0c, B->inv, v0c, st));
    const int ld = d + 1;
    const long pstride = (long)ld * d;
    double *Hs = nullptr;
    PP_TRY(dev_alloc(&Hs, (size_t)B->nsys * pstride));
    struct Free {
        double *p;
        ~Free() { dev_free(p); }
    } fh{Hs};
    HIP_TRY(hipMemsetAsync(Hs, 0, sizeof(double) * B->nsys * pstride, st));
    for (int j = 0; j < d; ++j) {
        void *bufs[5] = {bcol(w, prec, j), bcol(w, prec, j + 1), w.P(0), w.P(1), w.P(2)};
        HIP_TRY(launch_bchain(B->sell(prec), prec, R, B->desc_spmv, 1, 0, bufs, st));
        PP_TRY(bcgs2(B, prec, R, w, j, Hs + (size_t)j * ld, pstride, st));
    }
    std::vector<double> H((size_t)B->nsys * pstride);
    HIP_TRY(hipMemcpyAsync(H.data(), Hs, sizeof(double) * H.size(), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    std::vector<pp_poly> made;
    pp_status worst = PP_OK;
    for (int s = 0; s < B->nsys; ++s) {
        const double *Hb = H.data() + (size_t)s * pstride;
        int k = d;
        bool brk = false;
        double fro2 = 0.0;
        for (int j = 0; j < d; ++j) {
            for (int i = 0; i <= j + 1; ++i) fro2 += Hb[i + (size_t)j * ld] * Hb[i + (size_t)j * ld];
            if (!std::isfinite(fro2)) {
                for (auto p : made) delete p;
                set_error("pp_batch_setup: non-finite Hessenberg entry");
                return PP_EINVAL;
            }
            if (Hb[(j + 1) + (size_t)j * ld] <= kBreakdownTolB * std::sqrt(fro2)) {
                k = j + 1;
                brk = true;
                break;
            }
        }
        std::vector<double> hk((size_t)(k + 1) * k);
        for (int j = 0; j < k; ++j)
            for (int i = 0; i <= k; ++i) hk[i + (size_t)j * (k + 1)] = Hb[i + (size_t)j * ld];
        std::vector<double> re(k), im(k);
        int hs = harmonic_ritz(k, hk.data(), brk, re.data(), im.data());
        auto *p = hs == PP_OK ? new (std::nothrow) pp_poly_s() : nullptr;
        if (hs == PP_OK && !p) hs = PP_ENOMEM;
        if (hs == PP_OK) hs = plan_roots(k, re.data(), im.data(), add_roots != 0, p->plan);
        if (hs != PP_OK) {
            delete p;
            for (auto q : made) delete q;
            set_error("pp_batch_setup: system " + std::to_string(s) + ": harmonic Ritz values failed");
            return (pp_status)(hs < 0 ? hs : PP_ESINGULAR);
        }
        p->theta_re = re;
        p->theta_im = im;
        p->breakdown = brk ? 1 : 0;
        p->finalize();
        made.push_back(p);
        if (brk && k < d) worst = PP_BREAKDOWN;
        if (infos) {
            infos[s].d = k;
            infos[s].d_eff = p->plan.d_eff;
            infos[s].n_added = p->plan.n_added;
            infos[s].breakdown = brk ? 1 : 0;
            infos[s].mvps = k;
            infos[s].dots = (int64_t)k * (k + 2);
            infos[s].t_setup_s = now_s() - t0;
        }
    }
    for (int s = 0; s < B->nsys; ++s) polys[s] = made[s];
    return worst;
}

pp_status pp_batch_solve(pp_batch B, const pp_poly *polys, int nrhs, const double *b, double *x,
                         const pp_solve_opts *opts, void *stream, pp_info *infos) {
    if (!B || !polys || !b || !x || !opts || !(nrhs == 1 || nrhs == 2 || nrhs == 4) || opts->m < 1 ||
        opts->max_cycles < 0 || !(opts->tol > 0.0) || opts->inner < 0 || opts->inner > 2 ||
        opts->new_poly_degree != 0) {
        set_error("pp_batch_solve: bad argument (nrhs must be 1, 2 or 4; no new polynomial per cycle)");
        return PP_EINVAL;
    }
    // the kernels move the nrhs values of a row as one vector access
    const uintptr_t al = (uintptr_t)(8 * nrhs);
    if ((uintptr_t)b % al != 0 || (uintptr_t)x % al != 0) {
        set_error("pp_batch_solve: b and x must be aligned to nrhs doubles (8*nrhs bytes)");
        return PP_EINVAL;
    }
    for (int s = 0; s < B->nsys; ++s)
        if (!polys[s] || polys[s]->inner) {
            set_error("pp_batch_solve: null or composite polynomial");
            return PP_EINVAL;
        }
    hipStream_t st = S(stream);
    if (opts->graphs) {
        // the solve runs on the batch's own stream, after the caller's work
        if (!B->gstream) {
            HIP_TRY(hipStreamCreateWithFlags(&B->gstream, hipStreamNonBlocking));
            HIP_TRY(hipEventCreateWithFlags(&B->gevent, hipEventDisableTiming));
        }
        HIP_TRY(hipEventRecord(B->gevent, st));
        HIP_TRY(hipStreamWaitEvent(B->gstream, B->gevent, 0));
        st = B->gstream;
    }
    // whatever the exit, the solve's stream is drained before returning
    struct Drain {
        hipStream_t s;
        bool own;
        ~Drain() {
            if (own) (void)hipStreamSynchronize(s);
        }
    } drain{st, opts->graphs != 0};
    const double t0 = now_s();
    const int R = nrhs, m = opts->m;
    const int P = B->nsys * R;
    const long nR = B->n * R;
    PP_TRY(B->ensure_red(m + 1, R));
    PP_TRY(B->ensure(opts->inner, m, R));
    if (!B->cfg[opts->inner][R].tuned) PP_TRY(tune_bchain(B, opts->inner, R, st));
    const BatchBlocks bl = B->blocks();
    BatchProg phi, pol;
    PP_TRY(upload_programs(B, polys, PP_APPLY_PHI, phi, st));
    PP_TRY(upload_programs(B, polys, PP_APPLY_P, pol, st));
    std::vector<pp_info> inf(P);
    for (auto &i : inf) {
        std::memset(&i, 0, sizeof(i));
        i.relres_shortcut = NAN;
    }
    std::vector<double> bnorm, beta, beta_new;
    PP_TRY(bnorms(B, R, b, bnorm, st));
    HIP_TRY(launch_fill((int)nR, 0.0, x, st));
    HIP_TRY(hipMemcpyAsync(B->r64, b, sizeof(double) * nR, hipMemcpyDeviceToDevice, st));
    beta = bnorm;
    std::vector<char> done(P, 0), noconv(P, 0);
    std::vector<std::vector<double>> hist(P);
    int prec = opts->inner;
    int cycles = 0;
    PP_TRY(B->ensure_givens(m, R));
    const BGivens G = B->givens(R);
    double *gbeta = B->gin, *ginv = B->gin + 2 * P;
    // The device work of one restart cycle runs in segments of `seg`
    // Arnoldi steps, with no host synchronisation and no memset inside a
    // segment: the first segment takes the per-pair inputs in (from pinned
    // memory, read when the copy runs) and forms V0 = r / beta; every step
    // runs the phi chain, CGS2 and the Givens update of every running pair
    // (the masked kernels skip systems whose pairs have all stopped); each
    // segment ends by copying out whether some pair still runs, and the host
    // skips the rest of the cycle when none does. The tail forms z, the
    // correction x += p(A) V z and the true FP64 residual, and copies the
    // per-pair results out. With opts->graphs each segment and the tail are
    // captured once per precision into HIP graphs and replayed.
    const int seg = opts->graph_steps > 0 ? std::min(opts->graph_steps, m) : m;
    // two basis sweeps per step (delayed Gram-Schmidt) or three (CGS2)
    const bool delayed = B->orth == 1 && m <= bdcgs_max_cols();
    const int nseg = (m + seg - 1) / seg;
    auto segment_work = [&](int pr, int c) -> pp_status {
        const BWork &w = B->ws[pr];
        if (c == 0) {
            HIP_TRY(hipMemcpyAsync(B->gin, B->ginpin, sizeof(double) * 3 * P, hipMemcpyHostToDevice, st));
            HIP_TRY(hipMemcpyAsync(B->grun, B->grunpin, sizeof(int) * P, hipMemcpyHostToDevice, st));
            HIP_TRY(launch_bgivens_init(G, gbeta, st));
            // the first basis vector r / beta: column 0, or the first pending vector
            HIP_TRY(launch_bscale(bl, 0, pr, R, B->r64, ginv, delayed ? w.P(3) : bcol(w, pr, 0), st));
        }
        for (int j = c * seg; j < std::min(m, (c + 1) * seg); ++j) {
            if (delayed) {
                // phi(A) of the pending vector; its column completes one step later
                PP_TRY(run_bprog(B, pr, R, phi, w.P(3), bcol(w, pr, j + 1), w, st, true));
                PP_TRY(bdcgs(B, pr, R, w, j, false, st));
                if (j >= 1)
                    HIP_TRY(launch_bgivens_step(G, j - 1, B->dH + (size_t)(j - 1) * (m + 1), m * (m + 1),
                                                kBreakdownTolB, st));
                continue;
            }
            PP_TRY(run_bprog(B, pr, R, phi, bcol(w, pr, j), bcol(w, pr, j + 1), w, st, true));
            PP_TRY(bcgs2(B, pr, R, w, j, B->Hc, B->ldh, st, true));
            HIP_TRY(launch_bgivens_step(G, j, B->Hc, B->ldh, kBreakdownTolB, st));
        }
        HIP_TRY(launch_bany(B->act, B->nsys, B->gany, st));
        HIP_TRY(hipMemcpyAsync(B->ganypin, B->gany, sizeof(int), hipMemcpyDeviceToHost, st));
        return PP_OK;
    };
    auto tail_work = [&](int pr) -> pp_status {
        const BWork &w = B->ws[pr];
        if (delayed) {
            // the last column of the cycle: masked, so a no-op once no pair runs
            PP_TRY(bdcgs(B, pr, R, w, m, true, st));
            HIP_TRY(launch_bgivens_step(G, m - 1, B->dH + (size_t)(m - 1) * (m + 1), m * (m + 1), kBreakdownTolB,
                                        st));
        }
        HIP_TRY(launch_bgivens_solve(G, B->z, B->ldh, st));
        HIP_TRY(launch_bcombine(bl, pr, R, w.V, w.ldv, B->kdev, B->z, B->ldh, w.P(3), st));
        PP_TRY(run_bprog(B, pr, R, pol, w.P(3), w.P(4), w, st));
        HIP_TRY(launch_axpy_x(pr, (int)nR, 1.0, w.P(4), x, st));
        {
            const BWork &w64 = B->ws[0].V ? B->ws[0] : w;
            void *bufs[5] = {x, B->r64, (void *)b, w64.P(0), w64.P(1)};
            HIP_TRY(launch_bchain(B->sell(0, false, R), 0, R, B->desc_res, 1, 0, bufs, st));
        }
        HIP_TRY(hipMemcpyAsync(B->kpin, B->kdev, sizeof(int) * P, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipMemcpyAsync(B->gstepspin, B->gsteps, sizeof(int) * P, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipMemcpyAsync(B->gscpin, B->gsc, sizeof(double) * P, hipMemcpyDeviceToHost, st));
        return PP_OK;
    };
    // graphs per precision: segments 0 .. nseg-1, then the tail
    struct CycleGraphs {
        std::vector<hipGraphExec_t> ex;
        ~CycleGraphs() {
            for (auto e : ex)
                if (e) (void)hipGraphExecDestroy(e);
        }
    } graphs;
    graphs.ex.assign((size_t)3 * (nseg + 1), nullptr);
    auto run_part = [&](int pr, int part) -> pp_status {
        auto work = [&]() -> pp_status { return part < nseg ? segment_work(pr, part) : tail_work(pr); };
        if (!opts->graphs) return work();
        hipGraphExec_t &ex = graphs.ex[(size_t)pr * (nseg + 1) + part];
        if (!ex) {
            hipGraph_t g = nullptr;
            HIP_TRY(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
            const pp_status sw = work();
            const hipError_t ec = hipStreamEndCapture(st, &g);
            if (sw != PP_OK) {
                if (ec == hipSuccess && g) (void)hipGraphDestroy(g);
                return sw;
            }
            HIP_TRY(ec);
            const hipError_t ei = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
            (void)hipGraphDestroy(g);
            HIP_TRY(ei);
        }
        HIP_TRY(hipGraphLaunch(ex, st));
        return PP_OK;
    };
    for (int p = 0; p < P; ++p) B->gscpin[p] = NAN;
    for (;;) {
        int active = 0;
        for (int p = 0; p < P; ++p) {
            if (done[p]) continue;
            const double rel = bnorm[p] > 0 ? beta[p] / bnorm[p] : 0.0;
            hist[p].push_back(rel);
            inf[p].relres = rel;
            const int sc = opts->stall_cycles;
            if (rel <= opts->tol || !std::isfinite(rel)) {
                done[p] = 1;
                noconv[p] = !std::isfinite(rel);
            } else if (cycles >= opts->max_cycles ||
                       (sc > 0 && (int)hist[p].size() > sc && hist[p].back() > 0.99 * hist[p][hist[p].size() - 1 - sc])) {
                done[p] = 1;
                noconv[p] = 1;
            } else {
                ++active;
            }
        }
        if (active == 0) break;
        ++cycles;
        if (prec == PP_F64) {
            PP_TRY(B->ensure(0, m, R));
            if (!B->cfg[0][R].tuned) PP_TRY(tune_bchain(B, 0, R, st));
        }
        PP_TRY(upload_segments(B, polys, PP_APPLY_PHI, prec, R, phi, st));
        PP_TRY(upload_segments(B, polys, PP_APPLY_P, prec, R, pol, st));
        const double eta = (prec != PP_F64 && opts->inner_eta > 0.0) ? opts->inner_eta : kInnerEtaB[prec];
        // per-pair inputs of the cycle: beta, the inner target, 1/beta (0 for
        // pairs that are done) and the run flags
        for (int p = 0; p < P; ++p) {
            B->ginpin[p] = done[p] ? 0.0 : beta[p];
            B->ginpin[P + p] = std::max(opts->tol * bnorm[p], eta * beta[p]);
            B->ginpin[2 * P + p] = done[p] ? 0.0 : 1.0 / beta[p];
            B->grunpin[p] = done[p] ? 0 : 1;
            inf[p].cycles += done[p] ? 0 : 1;
            if (!done[p] && prec == PP_F64) inf[p].fp64_cycles++;
        }
        for (int c = 0; c < nseg; ++c) {
            PP_TRY(run_part(prec, c));
            if (c + 1 < nseg) {
                HIP_TRY(hipStreamSynchronize(st));
                if (!*B->ganypin) break;  // every pair has stopped: the rest of the cycle is skipped
            }
        }
        PP_TRY(run_part(prec, nseg));
        PP_TRY(bnorms(B, R, B->r64, beta_new, st));  // synchronises: the cycle's results are on the host
        bool stalled = false;
        for (int p = 0; p < P; ++p) {
            if (done[p]) continue;
            const int64_t st_p = B->gstepspin[p];
            const int64_t d_eff = polys[p / R]->plan.d_eff;
            inf[p].iters += (int)st_p;
            inf[p].mvps += st_p * d_eff + d_eff;  // the steps' phi chains; p(A) (d_eff - 1) and the residual (1)
            inf[p].dots += st_p * st_p + 2 * st_p;
            if (B->kpin[p] > 0) inf[p].relres_shortcut = B->gscpin[p] / bnorm[p];
            if (!(beta_new[p] <= 0.5 * beta[p])) stalled = true;
            beta[p] = beta_new[p];
        }
        if (prec != PP_F64 && stalled) prec = PP_F64;
    }
    pp_status status = PP_OK;
    const double t = now_s() - t0;
    for (int p = 0; p < P; ++p) {
        inf[p].status = noconv[p] ? PP_NOCONV : PP_OK;
        inf[p].t_solve_s = t;
        if (noconv[p]) status = PP_NOCONV;
        if (opts->history && p == 0)
            for (size_t i = 0; i < hist[p].size() && (int)i < opts->history_cap; ++i) opts->history[i] = hist[p][i];
    }
    if (infos)
        for (int p = 0; p < P; ++p) infos[p] = inf[p];
    return status;
}

}  // extern "C"
