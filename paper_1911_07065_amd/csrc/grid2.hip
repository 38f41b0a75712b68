// 2-D multi-step chain kernel of one matrix: k_grid2 and its launcher.
#include "grid2.h"

#include <cstdint>

#include "grid2_core.h"

namespace ppg {
namespace {

template <typename AT>
struct G2Args {
    const AT *in;
    AT *out;
    AT *acc;
    const AT *vfin;
    const AT *coef;
    const AT *dval;
    int gx, gy, hx, hy, tx, ty, ntx, ntiles;
    int n, load_acc, remap;
    Grid2Step<AT> steps[kGrid2MaxSteps];
};

// Tile t delivers tx x ty points after n steps from a region that is hx, hy
// = RHO n points wider on each side (0 where the region spans the grid).
//
// What bounds it: per step the issue of the region's operations (10 a point
// for 5 diagonals in FP64, 7 of them FP64) and one barrier, per launch 3.6 us
// for the launch and the trips to memory. Measured per step, against the best
// of one to four steps per launch through memory and LDS planes: FP64 50^2
// 0.6 us (2.5), 512^2 0.86 us (3.3), 1024^2 1.40 us (4.4), per-row values
// on 600 x 431 1.0 us (5.1), 13 points on 200^2 1.2 us (4.1); FP32 1024^2
// 1.13 us.
template <typename AT, int ND, bool VAR, int VX, int RY>
__global__ __launch_bounds__(1024) void k_grid2(G2Args<AT> a) {
    using G = Grid2<AT, ND, VAR, VX, 1, RY>;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, waves = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t = remap_tile(blockIdx.x, a.ntiles, a.remap);
    const int gx = a.gx, gy = a.gy;
    const int x0 = (t % a.ntx) * a.tx, y0 = (t / a.ntx) * a.ty;  // the tile
    const int x = x0 - a.hx + lane * VX, yw = y0 - a.hy + wave * RY;
    const bool all = x0 - a.hx >= 0 && x0 - a.hx + 64 * VX <= gx && y0 - a.hy >= 0 && y0 - a.hy + waves * RY <= gy;
    typename G::Rows A, B;
    typename G::AccRows acc;
    typename G::Coef cf;
    typename G::Live live;
    Grid2Step<AT> mine = a.steps[min(lane, a.n - 1)];
    // every load before the first use: the input, the accumulator or the
    // final vector (never both), per-row coefficients
    const bool has_side = a.vfin || a.load_acc;
    const AT *side = a.vfin ? a.vfin : (a.load_acc ? a.acc : a.in);
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const long line = (long)min(max(yw + r, 0), gy - 1) * gx;
        line_load<AT, VX>(a.in + line, x, gx, A[r]);
        line_load<AT, VX>(side + line, x, gx, acc[r]);
    }
    if constexpr (VAR) {
#pragma unroll
        for (int r = 0; r < RY; ++r)
#pragma unroll
            for (int v = 0; v < VX; ++v) {
                const long i = (long)min(max(yw + r, 0), gy - 1) * gx + min(max(x + v, 0), gx - 1);
                const AT *p = a.dval + (i >> 8) * ND * 256 + (i & 255);
#pragma unroll
                for (int d = 0; d < ND; ++d) cf[r * VX + v][d] = p[d * 256];
            }
    } else {
#pragma unroll
        for (int d = 0; d < ND; ++d) cf[0][d] = a.coef[d];
    }
#pragma unroll
    for (int r = 0; r < RY; ++r)
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            loaded(A[r][v]);
            loaded(acc[r][v]);
        }
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = yw + r;
        const bool in = y >= 0 && y < gy;
        line_pick<AT, VX>(x, gx, in, A[r]);
        line_pick<AT, VX>(x, gx, in && has_side, acc[r]);
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            B[r][v] = AT(0);
            live[r][v] = in && x + v >= 0 && x + v < gx;
        }
    }
    G::run_any(A, B, acc, a.n, mine, cf, reinterpret_cast<AT *>(smem), wave, waves, lane, all, a.acc != nullptr, live);
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        const int y = yw + r;
        if (y < y0 || y >= min(y0 + a.ty, gy)) continue;
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            if (x + v < x0 || x + v >= min(x0 + a.tx, gx)) continue;
            const long i = (long)y * gx + x + v;
            if (a.acc) a.acc[i] = acc[r][v];
            if (a.out) a.out[i] = a.vfin ? acc[r][v] - A[r][v] : A[r][v];
        }
    }
}

template <typename AT, int ND, bool VAR, int VX, int RY>
hipError_t g2_launch(const G2Args<AT> &a, const Grid2Shape &s, hipStream_t st) {
    using G = Grid2<AT, ND, VAR, VX, 1, RY>;
    const size_t lds = G::lds_values(s.waves) * sizeof(AT);
    if (lds > 64 * 1024) {  // per device, and cheap next to such a launch
        const hipError_t e = hipFuncSetAttribute((const void *)&k_grid2<AT, ND, VAR, VX, RY>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_grid2<AT, ND, VAR, VX, RY>), dim3((unsigned)a.ntiles), dim3(64 * s.waves), lds, st, a);
    return hipGetLastError();
}

// The built shapes (grid2_built): one column of 2, 3, 4 or 6 rows a lane, or
// two of 2, 3 or 4. One row a wave pays the barrier for too little work and
// 12 or 16 points a lane (8 waves, their registers) gain nothing: at 1024^2 in FP64
// 1.41 us a step with 2 x 4, 1.49 with 2 x 8 (2 x 4 in FP64 spills 4 vector
// registers of its 128, with 13 points 18; the tuner times it like the
// others). Per-row coefficients stay in registers, 5 a point, so those stop
// at 4 points a lane.
template <typename AT, int ND, bool VAR>
hipError_t g2_shape(const G2Args<AT> &a, const Grid2Shape &s, hipStream_t st) {
    switch (s.vx * 10 + s.ry) {
        case 12: return g2_launch<AT, ND, VAR, 1, 2>(a, s, st);
        case 13: return g2_launch<AT, ND, VAR, 1, 3>(a, s, st);
        case 14: return g2_launch<AT, ND, VAR, 1, 4>(a, s, st);
        case 22: return g2_launch<AT, ND, VAR, 2, 2>(a, s, st);
    }
    if constexpr (!VAR) {
        if (s.vx == 1 && s.ry == 6) return g2_launch<AT, ND, VAR, 1, 6>(a, s, st);
        if (s.vx == 2 && s.ry == 3) return g2_launch<AT, ND, VAR, 2, 3>(a, s, st);
        if (s.vx == 2 && s.ry == 4) return g2_launch<AT, ND, VAR, 2, 4>(a, s, st);
    }
    return hipErrorInvalidValue;
}

template <typename AT>
hipError_t g2_dispatch(const G2Args<AT> &a, const Grid2Mat &m, const Grid2Shape &s, hipStream_t st) {
    if (m.nd == 13) return g2_shape<AT, 13, false>(a, s, st);
    return m.constant() ? g2_shape<AT, 5, false>(a, s, st) : g2_shape<AT, 5, true>(a, s, st);
}

template <typename AT>
hipError_t g2_run(const Grid2Mat &m, const AT *coef, const AT *dval, const Grid2Shape &s, const Grid2Ptrs &p,
                  int remap, hipStream_t st) {
    G2Args<AT> a;
    long tiles = 0;
    if (p.n < 1 || p.n > kGrid2MaxSteps || !grid2_tiles(m.form(), s, p.n, &a.tx, &a.ty, &tiles) || tiles >= (1L << 31) ||
        (m.constant() ? !coef : !dval))
        return hipErrorInvalidValue;
    a.in = (const AT *)p.in;
    a.out = (AT *)p.out;
    a.acc = (AT *)p.acc;
    a.vfin = (const AT *)p.vfin;
    a.coef = coef;
    a.dval = dval;
    a.gx = m.gx;
    a.gy = m.gy;
    a.hx = a.tx == m.gx ? 0 : m.rho() * p.n;
    a.hy = a.ty == m.gy ? 0 : m.rho() * p.n;
    a.ntx = (m.gx + a.tx - 1) / a.tx;
    a.ntiles = (int)tiles;
    a.n = p.n;
    a.load_acc = p.acc ? p.load_acc : 0;
    a.remap = remap;
    if (p.acc && p.vfin) return hipErrorInvalidValue;
    for (int k = 0; k < p.n; ++k) {
        const Grid2Step<double> &u = p.steps[k];
        const int unit = u.a1 == 1.0 && !(u.flags & kG2Aux) ? kG2Unit : 0;
        a.steps[k] = Grid2Step<AT>{(AT)u.a0, (AT)u.a1, (AT)u.a2, (AT)u.b0, (AT)u.b1, u.flags | unit};
    }
    return g2_dispatch<AT>(a, m, s, st);
}

}  // namespace

hipError_t launch_chain_grid2(const Grid2Mat &m, int prec, const Grid2Shape &s, const Grid2Ptrs &p, int remap,
                              hipStream_t st) {
    if (!grid2_built(m, prec, s.vx, s.ry)) return hipErrorInvalidValue;
    if (prec == 0) return g2_run<double>(m, m.coef64, m.dval64, s, p, remap, st);
    return g2_run<float>(m, m.coef32, m.dval32, s, p, remap, st);
}

}  // namespace ppg
