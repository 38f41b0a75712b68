// Many chain steps per launch of a batch of 2-D grid stencils: k_bgrid and
// its launcher.
#include "batched.h"
#include "grid2_core.h"

namespace ppg {
namespace {

template <typename AT>
struct BGArgs {
    const int4 *tile;
    int ntiles, halo, ry_waves, remap;
    const int *active;
    const PStep *desc;
    const BatchSeg *segs;
    int K, L, l;
    AT *bufs[5];
    const int32_t *bgx, *bpint, *ptoff, *sysoff;
    const AT *ptab;
};

// The R interleaved values of one row.
template <typename AT, int R>
struct RowVec {
    typedef AT T __attribute__((ext_vector_type(R)));
};
template <typename AT>
struct RowVec<AT, 1> {
    typedef AT T;
};

template <typename AT, int R>
__device__ __forceinline__ AT pick(const typename RowVec<AT, R>::T &v, int c) {
    if constexpr (R == 1)
        return v;
    else
        return v[c];
}

// Tile t.{y, z} (its first column and row in system t.x's grid) of launch l:
// the segment of the system's own program on a region of 64 x waves RY
// points, R values a point, as k_grid2 runs one matrix. The tile is what a
// launch of `halo` steps leaves exact; shorter segments use the same tiles.
//
// What bounds it: the issue of the region's operations (8 a value in FP32)
// and, per launch, one read of the regions and one write of the tiles: 48
// systems of sides 64 to 256 with 4 right-hand sides in FP32 take 29.5 us for
// seven steps, 10.4 us a step in launches of one step, which move every
// vector through memory. ACC: a launch
// with an accumulator, a third vector in registers and so fewer waves; phi
// chains have none (their final vector is read at the end).
template <typename AT, int R, int RY, bool ACC>
__global__ __launch_bounds__(64 * batch_grid_max_waves(sizeof(AT), R, RY, ACC)) void k_bgrid(BGArgs<AT> a) {
    using G = Grid2<AT, 5, false, 1, R, RY, ACC>;
    using Vec = typename RowVec<AT, R>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    const int4 t = a.tile[remap_tile(blockIdx.x, a.ntiles, a.remap)];
    const int sys = t.x, x0 = t.y, y0 = t.z;
    if (!a.active[sys]) return;
    const BatchSeg seg = a.segs[(long)sys * a.L + a.l];
    if (seg.count == 0) return;
    const int lane = threadIdx.x & 63, waves = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int base = a.sysoff[sys], gx = a.bgx[sys], gy = (a.sysoff[sys + 1] - base) / gx;
    const int hx = gx <= 64 ? 0 : a.halo, hy = gy <= a.ry_waves ? 0 : a.halo;
    const int x1 = gx <= 64 ? gx : min(x0 + 64 - 2 * a.halo, gx);
    const int y1 = gy <= a.ry_waves ? gy : min(y0 + a.ry_waves - 2 * a.halo, gy);
    const int x = x0 - hx + lane, yw = y0 - hy + wave * RY;
    const bool all = x0 - hx >= 0 && x0 - hx + 64 <= gx && y0 - hy >= 0 && y0 - hy + a.ry_waves <= gy;
    const AT *in = a.bufs[seg.in], *fin = seg.fin ? a.bufs[0] : nullptr;
    AT *out = seg.out >= 0 ? a.bufs[seg.out] : nullptr, *accp = seg.acc >= 0 ? a.bufs[seg.acc] : nullptr;
    const bool load_acc = ACC && accp && !seg.acc_init;
    // lane k's step of the segment
    const PStep ps = a.desc[(long)sys * a.K + seg.first + min(lane, seg.count - 1)];
    const AT *cp = a.ptab + a.ptoff[sys] + (long)a.bpint[sys] * 5;
    typename G::Rows A, B;
    typename G::AccRows acc;
    typename G::Coef cf;
    typename G::Live live;
    Vec va[RY], vs[ACC ? RY : 1];
    const int xc = min(max(x, 0), gx - 1);
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const long i = base + (long)min(max(yw + r, 0), gy - 1) * gx + xc;
        va[r] = reinterpret_cast<const Vec *>(in)[i];
        if constexpr (ACC) vs[r] = reinterpret_cast<const Vec *>(load_acc ? accp : in)[i];
    }
#pragma unroll
    for (int d = 0; d < 5; ++d) cf[0][d] = cp[d];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = yw + r;
        live[r][0] = y >= 0 && y < gy && x >= 0 && x < gx;
#pragma unroll
        for (int c = 0; c < R; ++c) {
            A[r][c] = pick<AT, R>(va[r], c);
            loaded(A[r][c]);
            if constexpr (ACC) {
                acc[r][c] = pick<AT, R>(vs[r], c);
                loaded(acc[r][c]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RY; ++r)
#pragma unroll
        for (int c = 0; c < R; ++c) {
            A[r][c] = live[r][0] ? A[r][c] : AT(0);
            if constexpr (ACC) acc[r][c] = load_acc && live[r][0] ? acc[r][c] : AT(0);
            B[r][c] = AT(0);
        }
    Grid2Step<AT> mine{(AT)ps.a0, (AT)ps.a1, (AT)ps.a2, (AT)ps.b0, (AT)ps.b1, 0};
    mine.flags = ps.aux >= 0 ? kG2Aux : (ps.a1 == 1.0 ? kG2Unit : 0);
    G::run_any(A, B, acc, seg.count, mine, cf, reinterpret_cast<AT *>(smem), wave, waves, lane, all, ACC, live);
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = yw + r;
        if (y < y0 || y >= y1 || x < x0 || x >= x1) continue;
        const long i = base + (long)y * gx + x;
        Vec vf = fin ? reinterpret_cast<const Vec *>(fin)[i] : Vec(AT(0)), o, oa;
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const AT w = fin ? pick<AT, R>(vf, c) - A[r][c] : A[r][c];
            if constexpr (R == 1) {
                o = w;
                if constexpr (ACC) oa = acc[r][c];
            } else {
                o[c] = w;
                if constexpr (ACC) oa[c] = acc[r][c];
            }
        }
        if constexpr (ACC) reinterpret_cast<Vec *>(accp)[i] = oa;
        if (out) reinterpret_cast<Vec *>(out)[i] = o;
    }
}

template <typename AT, int R, int RY, bool ACC>
hipError_t bg_launch(const BGArgs<AT> &a, int waves, hipStream_t st) {
    if constexpr (batch_grid_max_waves(sizeof(AT), R, RY, ACC) > 0) {
        using G = Grid2<AT, 5, false, 1, R, RY, ACC>;
        if (waves > batch_grid_max_waves(sizeof(AT), R, RY, ACC)) return hipErrorInvalidValue;
        const size_t lds = G::lds_values(waves) * sizeof(AT);
        if (lds > 64 * 1024) {  // per device, and cheap next to such a launch
            const hipError_t e = hipFuncSetAttribute((const void *)&k_bgrid<AT, R, RY, ACC>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL((k_bgrid<AT, R, RY, ACC>), dim3((unsigned)a.ntiles), dim3(64 * waves), lds, st, a);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <typename AT, int R, bool ACC>
hipError_t bg_rows(const BGArgs<AT> &a, int ry, int waves, hipStream_t st) {
    switch (ry) {
        case 2: return bg_launch<AT, R, 2, ACC>(a, waves, st);
        case 3: return bg_launch<AT, R, 3, ACC>(a, waves, st);
        case 4: return bg_launch<AT, R, 4, ACC>(a, waves, st);
        case 6: return bg_launch<AT, R, 6, ACC>(a, waves, st);
    }
    return hipErrorInvalidValue;
}

template <typename AT>
hipError_t bg_run(const BatchSell &S, const AT *ptab, const BatchGrid &g, bool acc, int R, const PStep *desc, int K,
                  const BatchSeg *segs, int L, int l, void *const bufs[5], hipStream_t st) {
    BGArgs<AT> a;
    const int waves = acc ? g.acc_waves : g.waves;
    a.tile = acc ? g.acc_tile : g.tile;
    a.ntiles = acc ? g.acc_ntiles : g.ntiles;
    a.halo = g.steps;
    a.ry_waves = g.ry * waves;
    a.remap = 1;
    a.active = S.active;
    a.desc = desc;
    a.segs = segs;
    a.K = K;
    a.L = L;
    a.l = l;
    for (int k = 0; k < 5; ++k) a.bufs[k] = (AT *)bufs[k];
    a.bgx = S.bgx;
    a.bpint = S.bpint;
    a.ptoff = S.ptoff;
    a.sysoff = S.sysoff;
    a.ptab = ptab;
    if (!a.tile) return hipErrorInvalidValue;
    switch (R) {
        case 1: return acc ? bg_rows<AT, 1, true>(a, g.ry, waves, st) : bg_rows<AT, 1, false>(a, g.ry, waves, st);
        case 2: return acc ? bg_rows<AT, 2, true>(a, g.ry, waves, st) : bg_rows<AT, 2, false>(a, g.ry, waves, st);
        case 4: return acc ? bg_rows<AT, 4, true>(a, g.ry, waves, st) : bg_rows<AT, 4, false>(a, g.ry, waves, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_bgrid(const BatchSell &S, const BatchGrid &g, bool acc, int prec, int R, const PStep *desc, int K,
                        const BatchSeg *segs, int L, int l, void *const bufs[5], hipStream_t st) {
    if (!S.bgx || !batch_grid_ok(prec, R, g.ry, g.waves, g.steps)) return hipErrorInvalidValue;
    if ((acc ? g.acc_ntiles : g.ntiles) == 0) return hipSuccess;
    if (prec == 0) return bg_run<double>(S, S.ptab64, g, acc, R, desc, K, segs, L, l, bufs, st);
    return bg_run<float>(S, S.ptab32, g, acc, R, desc, K, segs, L, l, bufs, st);
}

}  // namespace ppg
