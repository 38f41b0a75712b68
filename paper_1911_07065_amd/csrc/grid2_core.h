// Device core of the 2-D multi-step chain kernels (internal): several steps of
// a chain program on one tile of a grid, everything between the first load
// and the last store held in registers.
#pragma once

#include <hip/hip_runtime.h>

#include "devutil.h"
#include "grid2.h"

namespace ppg {
namespace {

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// lane k's step, uniform in the wave
__device__ __forceinline__ float lane_value(float v, int k) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
__device__ __forceinline__ double lane_value(double v, int k) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                            __builtin_amdgcn_readlane(__double2loint(v), k));
}
template <typename AT>
__device__ __forceinline__ Grid2Step<AT> lane_step(const Grid2Step<AT> &s, int k) {
    return Grid2Step<AT>{lane_value(s.a0, k), lane_value(s.a1, k), lane_value(s.a2, k), lane_value(s.b0, k),
                         lane_value(s.b1, k), __builtin_amdgcn_readlane(s.flags, k)};
}

// Keeps loaded values where they are loaded: without it a load whose only
// use is a select sinks into a branch of its own and waits there alone.
__device__ __forceinline__ void loaded(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void loaded(double &v) { asm volatile("" : "+v"(v)); }

// VX adjacent points of a grid line (p, gx points) from column x: line_load
// reads them, line_pick drops what lies outside the line. Two columns are
// one access on an element-aligned address, moved inside the line and
// picked apart.
template <typename AT, int VX>
__device__ __forceinline__ void line_load(const AT *p, int x, int gx, AT *o) {
    if constexpr (VX == 1) {
        o[0] = p[min(max(x, 0), gx - 1)];
    } else {
        typedef AT Pair __attribute__((ext_vector_type(2), aligned(sizeof(AT))));
        const Pair t = *reinterpret_cast<const Pair *>(p + min(max(x, 0), gx - 2));
        o[0] = t[0];
        o[1] = t[1];
    }
}
template <typename AT, int VX>
__device__ __forceinline__ void line_pick(int x, int gx, bool in, AT *o) {
    if constexpr (VX == 1) {
        o[0] = in && x >= 0 && x < gx ? o[0] : AT(0);
    } else {
        const int xb = min(max(x, 0), gx - 2);
        const AT t0 = o[0], t1 = o[1];
        o[0] = in && x >= 0 && x < gx ? (x == xb ? t0 : t1) : AT(0);
        o[1] = in && x + 1 >= 0 && x + 1 < gx ? (x + 1 == xb ? t0 : t1) : AT(0);
    }
}

// A wave owns RY consecutive grid rows of 64 VX columns, a lane VX adjacent
// columns of them with NC interleaved values per point (NV = VX NC values a
// row). The column neighbours are lane moves, the row neighbours the lane's
// own registers, and only the outermost RHO rows of a wave travel through
// LDS: two buffers that alternate between steps, so one barrier a step.
// Values outside the tile's region read as zero; what that spoils moves
// inwards RHO points a step, which is why a region is RHO points wider per
// step than the tile it delivers, except where the region ends with the grid.
//
// ND 5: the stencil of the diagonals -g, -1, 0, 1, g; ND 13: of -2g, -g-1,
// -g, -g+1, -2, -1, 0, 1, 2, g-1, g, g+1, 2g. VAR: the coefficients are the
// lane's own (per point); otherwise one set for all points.
//
// WITH_ACC: launches may have an accumulator or a final vector, which is one
// more value a point in registers (acc); without it acc is not touched.
template <typename AT, int ND, bool VAR, int VX, int NC, int RY, bool WITH_ACC = true>
struct Grid2 {
    static_assert(ND == 5 || ND == 13, "5- or 13-point stencils");
    static constexpr int RHO = ND == 13 ? 2 : 1;
    static constexpr int NV = VX * NC;
    static constexpr int NSLOT = RY < 2 * RHO ? RY : 2 * RHO;  // rows a wave publishes
    static_assert(RY >= RHO, "a wave's edge rows are its own");
    static constexpr int NCOEF = VAR ? RY * VX : 1;
    typedef AT Rows[RY][NV];
    typedef AT AccRows[WITH_ACC ? RY : 1][WITH_ACC ? NV : 1];
    typedef AT Coef[NCOEF][ND];
    typedef bool Live[RY][VX];

    // LDS values of `waves` waves (both buffers)
    static constexpr size_t lds_values(int waves) { return (size_t)2 * waves * NSLOT * NV * 64; }

    // value v of a row DX columns to the left (DX < 0) or right
    template <int DX>
    static __device__ __forceinline__ AT shifted(const AT (&row)[NV], int v) {
        const int vx = v / NC, c = v % NC, q = vx + DX;
        if (q >= 0 && q < VX) return row[q * NC + c];
        if constexpr (DX < 0) {
            const int lanes = (-q + VX - 1) / VX;
            AT t = lane_left(row[(q + lanes * VX) * NC + c]);
            if (lanes == 2) t = lane_left(t);
            return t;
        } else {
            const int lanes = q / VX;
            AT t = lane_right(row[(q - lanes * VX) * NC + c]);
            if (lanes == 2) t = lane_right(t);
            return t;
        }
    }

    // what a step adds to a0 (A S): S alone (a real root: a1 = 1), a1 S, or
    // a1 S + a2 D with D's old values, the vector before S (a conjugate
    // pair's second step)
    enum Kind { UNIT, PLAIN, AUX };

    // One row of a step into D, up and dn the rows beyond the wave's own.
    // MASK: points that are not live (outside the grid) stay zero. Products
    // are summed in ascending diagonal order. KIND, ACC and MASK are
    // compile-time because a uniform test inside the row loop becomes
    // arithmetic on both sides and a select: 27 operations a point in FP64
    // instead of 10.
    template <bool MASK, bool ACC, int KIND>
    static __device__ __forceinline__ void row(int r, const Rows &S, Rows &D, AccRows &acc, const Grid2Step<AT> &s,
                                               const Coef &cf, const AT (&up)[RHO][NV], const AT (&dn)[RHO][NV],
                                               const Live &live) {
        const AT(&m1)[NV] = r >= 1 ? S[r >= 1 ? r - 1 : 0] : up[RHO - 1];
        const AT(&p1)[NV] = r + 1 < RY ? S[r + 1 < RY ? r + 1 : 0] : dn[0];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const AT *c = cf[VAR ? r * VX + v / NC : 0];
            AT t;
            if constexpr (ND == 5) {
                t = c[0] * m1[v];
                t += c[1] * shifted<-1>(S[r], v);
                t += c[2] * S[r][v];
                t += c[3] * shifted<1>(S[r], v);
                t += c[4] * p1[v];
            } else {
                const AT(&m2)[NV] = r >= 2 ? S[r >= 2 ? r - 2 : 0] : up[r < 2 ? r : 0];
                const AT(&p2)[NV] = r + 2 < RY ? S[r + 2 < RY ? r + 2 : 0] : dn[r + 2 < RY ? 0 : r + 2 - RY];
                t = c[0] * m2[v];
                t += c[1] * shifted<-1>(m1, v);
                t += c[2] * m1[v];
                t += c[3] * shifted<1>(m1, v);
                t += c[4] * shifted<-2>(S[r], v);
                t += c[5] * shifted<-1>(S[r], v);
                t += c[6] * S[r][v];
                t += c[7] * shifted<1>(S[r], v);
                t += c[8] * shifted<2>(S[r], v);
                t += c[9] * shifted<-1>(p1, v);
                t += c[10] * p1[v];
                t += c[11] * shifted<1>(p1, v);
                t += c[12] * p2[v];
            }
            AT w = fma_(s.a0, t, KIND == UNIT ? S[r][v] : s.a1 * S[r][v]);
            if (KIND == AUX) w = fma_(s.a2, D[r][v], w);
            if (MASK) w = live[r][v / NC] ? w : AT(0);
            if (ACC) acc[r][v] = fma_(s.b1, w, fma_(s.b0, S[r][v], acc[r][v]));
            D[r][v] = w;
        }
    }

    // D = a0 (A S) + ... (see Kind), acc += b0 S + b1 D. The rows that need
    // none of the neighbouring waves' are computed between the edge rows' way
    // into LDS and the barrier.
    template <bool MASK, bool ACC, int KIND>
    static __device__ __forceinline__ void step(const Rows &S, Rows &D, AccRows &acc, const Grid2Step<AT> &s,
                                                const Coef &cf, AT *edge, int wave, int waves, int lane,
                                                const Live &live) {
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            const bool top = r < RHO, bot = r >= RY - RHO;
            if (!top && !bot) continue;
            const int slot = top ? r : NSLOT - (RY - r);
#pragma unroll
            for (int v = 0; v < NV; ++v) edge[((wave * NSLOT + slot) * NV + v) * 64 + lane] = S[r][v];
        }
        AT up[RHO][NV] = {}, dn[RHO][NV] = {};
#pragma unroll
        for (int r = RHO; r < RY - RHO; ++r) row<MASK, ACC, KIND>(r, S, D, acc, s, cf, up, dn, live);
        __syncthreads();
        if (wave > 0) {
#pragma unroll
            for (int k = 0; k < RHO; ++k)
#pragma unroll
                for (int v = 0; v < NV; ++v)
                    up[k][v] = edge[(((wave - 1) * NSLOT + NSLOT - RHO + k) * NV + v) * 64 + lane];
        }
        if (wave + 1 < waves) {
#pragma unroll
            for (int k = 0; k < RHO; ++k)
#pragma unroll
                for (int v = 0; v < NV; ++v) dn[k][v] = edge[(((wave + 1) * NSLOT + k) * NV + v) * 64 + lane];
        }
#pragma unroll
        for (int r = 0; r < RY; ++r)
            if (r < RHO || r >= RY - RHO) row<MASK, ACC, KIND>(r, S, D, acc, s, cf, up, dn, live);
    }

    template <bool MASK, bool ACC>
    static __device__ __forceinline__ void any_step(const Rows &S, Rows &D, AccRows &acc, const Grid2Step<AT> &s,
                                                    const Coef &cf, AT *edge, int wave, int waves, int lane,
                                                    const Live &live) {
        if (s.flags & kG2Aux)
            step<MASK, ACC, AUX>(S, D, acc, s, cf, edge, wave, waves, lane, live);
        else if (s.flags & kG2Unit)
            step<MASK, ACC, UNIT>(S, D, acc, s, cf, edge, wave, waves, lane, live);
        else
            step<MASK, ACC, PLAIN>(S, D, acc, s, cf, edge, wave, waves, lane, live);
    }

    // Runs `n` steps from the vector in A; the result is left in A. B is
    // scratch, acc takes every step's update with ACC. Lane k of the wave
    // holds step k (every wave has its own copy: a lane read costs a few
    // cycles, a scalar load a memory round trip on every step's critical path).
    template <bool MASK, bool ACC>
    static __device__ __forceinline__ void run(Rows &A, Rows &B, AccRows &acc, int n, const Grid2Step<AT> &mine,
                                               const Coef &cf, AT *lds, int wave, int waves, int lane,
                                               const Live &live) {
        AT *e1 = lds + (size_t)waves * NSLOT * NV * 64;
        int k = 0;
        for (; k + 1 < n; k += 2) {
            any_step<MASK, ACC>(A, B, acc, lane_step(mine, k), cf, lds, wave, waves, lane, live);
            any_step<MASK, ACC>(B, A, acc, lane_step(mine, k + 1), cf, e1, wave, waves, lane, live);
        }
        if (k < n) {
            any_step<MASK, ACC>(A, B, acc, lane_step(mine, k), cf, lds, wave, waves, lane, live);
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int v = 0; v < NV; ++v) A[r][v] = B[r][v];
        }
    }

    // all: every point of the region lies inside the grid
    static __device__ __forceinline__ void run_any(Rows &A, Rows &B, AccRows &acc, int n, const Grid2Step<AT> &mine,
                                                   const Coef &cf, AT *lds, int wave, int waves, int lane, bool all,
                                                   bool with_acc, const Live &live) {
        if constexpr (WITH_ACC) {
            if (with_acc) {
                if (all)
                    run<false, true>(A, B, acc, n, mine, cf, lds, wave, waves, lane, live);
                else
                    run<true, true>(A, B, acc, n, mine, cf, lds, wave, waves, lane, live);
                return;
            }
        }
        if (all)
            run<false, false>(A, B, acc, n, mine, cf, lds, wave, waves, lane, live);
        else
            run<true, false>(A, B, acc, n, mine, cf, lds, wave, waves, lane, live);
    }
};

}  // namespace
}  // namespace ppg
