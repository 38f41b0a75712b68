// 3-D multi-step chain kernel of one matrix: k_grid3 and its launcher.
#include "grid3.h"

#include <algorithm>
#include <cstdint>

#include "grid2_core.h"

namespace ppg {
namespace {

// Threads of the largest workgroup: 1024 where a plane's values take at most
// four registers a lane (128 registers hold the march then), otherwise 512.
constexpr int grid3_threads(int value_bytes, int vx, int ry) { return value_bytes * vx * ry <= 16 ? 1024 : 512; }

template <typename AT>
struct G3Args {
    const AT *in;
    AT *out;
    AT *acc;
    const AT *vfin;
    const AT *coef;
    int gx, gy, gz, hx, hy, tx, ty, tz, ntx, nty, ntiles;
    int load_acc, remap;
    Grid2Step<AT> steps[kGrid3MaxSteps];
};

// What a launch has besides its input and output: nothing, an accumulator
// (the output may be absent), or the vector the last step is subtracted from.
enum Side { NONE, ACC, FIN };

// A workgroup marches through the planes of its region (64 VX columns, RY
// rows a wave) with S steps in flight, level l one plane behind level l - 1:
// iteration t reads plane t of the input and forms plane t - l of level l
// from planes t - l - 1 .. t - l + 1 of the level below. All of that stays in
// registers, the plane neighbours in the lane itself; columns come by lane
// moves and the rows beyond a wave through LDS, where every level publishes
// its new plane's outermost rows for the next iteration: two buffers in turn,
// one barrier an iteration. Planes lie in rings of four, so an iteration's
// slots depend on its phase alone, and four phases make up the loop. Points outside the
// region read as zero; what that spoils moves inwards a point a level, so
// the region is S points wider than its tile where it does not end with the
// grid, and each chunk of planes starts and ends S planes further out.
template <typename AT, int S, int VX, int RY, int SIDE>
struct March3 {
    using G = Grid2<AT, 5, false, VX, 1, RY>;
    typedef AT Plane[RY][VX];
    // plane t - k of the iteration t with phase PH lies in slot (PH - k) & 3
    Plane L[S][4];
    Plane C[SIDE != NONE ? 4 : 1];
    AT cf[7];
    unsigned off[RY];          // the lane's byte offset in a plane, clamped to the grid
    int back;                  // columns that the clamp moved the lane's pair back by
    bool live[RY][VX];         // the point lies inside the grid
    unsigned deliver;          // bit r VX + v: the point belongs to the tile
    int wave, waves, lane;

    // Plane z of the vector at p, as an address the compiler cannot take apart:
    // it would keep p + off[r] of every vector in registers otherwise.
    typedef __attribute__((address_space(1))) char *Global;
    static __device__ __forceinline__ Global plane(const AT *p, const G3Args<AT> &a, int z) {
        Global q = (Global)(p + (size_t)z * a.gx * a.gy);
        asm volatile("" : "+s"(q));
        return q;
    }
    template <typename T>
    static __device__ __forceinline__ __attribute__((address_space(1))) T &at(Global q, unsigned off) {
        asm volatile("" : "+v"(off));
        return *(__attribute__((address_space(1))) T *)(q + off);
    }
    __device__ __forceinline__ void load(const AT *p, const G3Args<AT> &a, int z, Plane &o) const {
        const Global q = plane(p, a, z);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            if constexpr (VX == 1) {
                o[r][0] = at<AT>(q, off[r]);
            } else {
                typedef AT Pair __attribute__((ext_vector_type(2), aligned(sizeof(AT))));
                const Pair t = at<Pair>(q, off[r]);
                o[r][0] = t[0];
                o[r][1] = t[1];
            }
        }
    }
    // drops what a load read for points outside the grid
    __device__ __forceinline__ void pick(const G3Args<AT> &a, bool in, Plane &o) const {
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            if constexpr (VX == 1) {
                o[r][0] = in && live[r][0] ? o[r][0] : AT(0);
            } else {
                const AT t0 = o[r][0], t1 = o[r][1];
                o[r][0] = in && live[r][0] ? (back ? t1 : t0) : AT(0);
                o[r][1] = in && live[r][1] ? (back ? t0 : t1) : AT(0);
            }
        }
    }
    // Step l, read from the kernel's arguments where it is used: with an
    // accumulator in FP64, three steps kept in scalar registers are spilled to
    // lanes and read back value by value (49 registers, 4 to 13 so; 201 x 150
    // x 97 p 8.6 us a step, 8.5 so; 50^3 2.75 and 2.64). FP32 with an
    // accumulator spills 18 to 35 with three steps, but ran no faster with
    // the reads, and forms without one, which hardly spill, 1 % slower.
    static constexpr bool kReread = SIDE == ACC && sizeof(AT) == 8;
    static __device__ __forceinline__ Grid2Step<AT> step_args(int l) {
        typedef __attribute__((address_space(4))) const char *Args;
        Args q = (Args)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(G3Args<AT>, steps) + l * sizeof(Grid2Step<AT>);
        asm volatile("" : "+s"(q));
        typedef __attribute__((address_space(4))) const Grid2Step<AT> *Steps;
        const Steps p = (Steps)q;
        return Grid2Step<AT>{p->a0, p->a1, p->a2, p->b0, p->b1, p->flags};
    }
    // edge rows of level l's plane in buffer b
    __device__ __forceinline__ AT *edge(AT *lds, int b, int l, int w, int bottom) const {
        return lds + ((((size_t)(b * S + l) * waves + w) * 2 + bottom) * VX) * 64 + lane;
    }
    __device__ __forceinline__ void publish(AT *lds, int b, int l, const Plane &p) const {
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            edge(lds, b, l, wave, 0)[v * 64] = p[0][v];
            edge(lds, b, l, wave, 1)[v * 64] = p[RY - 1][v];
        }
    }
    // w = a0 (A c) + a1 c [+ a2 aux], acc += b0 c + b1 w, for the plane c
    // between zm and zp; up and dn the rows beyond the wave's. Products are
    // summed in ascending diagonal order.
    template <int KIND>
    __device__ __forceinline__ void level(const Plane &zm, const Plane &c, const Plane &zp, const Plane &aux,
                                          const AT (&up)[VX], const AT (&dn)[VX], const Grid2Step<AT> &s, Plane &acc,
                                          Plane &w) const {
#pragma unroll
        for (int r = 0; r < RY; ++r) {
#pragma unroll
            for (int v = 0; v < VX; ++v) {
                AT t = cf[0] * zm[r][v];
                t += cf[1] * (r ? c[r ? r - 1 : 0][v] : up[v]);
                t += cf[2] * G::template shifted<-1>(c[r], v);
                t += cf[3] * c[r][v];
                t += cf[4] * G::template shifted<1>(c[r], v);
                t += cf[5] * (r + 1 < RY ? c[r + 1 < RY ? r + 1 : 0][v] : dn[v]);
                t += cf[6] * zp[r][v];
                AT u = fma_(s.a0, t, KIND == G::UNIT ? c[r][v] : s.a1 * c[r][v]);
                if (KIND == G::AUX) u = fma_(s.a2, aux[r][v], u);
                u = live[r][v] ? u : AT(0);
                if (SIDE == ACC) acc[r][v] = fma_(s.b1, u, fma_(s.b0, c[r][v], acc[r][v]));
                w[r][v] = u;
            }
        }
    }
    template <int PH, int LV>
    __device__ __forceinline__ void advance(const G3Args<AT> &a, AT *lds, int t, int lo, int hi) {
        // planes lo .. hi - 1 of level LV are needed and lie in the grid; others are zero
        constexpr int zp = (PH - LV + 1) & 3, c = (PH - LV) & 3, zm = (PH - LV - 1) & 3;
        const int z = t - LV;
        Plane w;
        if (z >= lo && z < hi) {
            AT up[VX], dn[VX];
            const int wu = max(wave - 1, 0), wd = min(wave + 1, waves - 1);
#pragma unroll
            for (int v = 0; v < VX; ++v) {
                up[v] = edge(lds, (PH & 1) ^ 1, LV - 1, wu, 1)[v * 64];
                dn[v] = edge(lds, (PH & 1) ^ 1, LV - 1, wd, 0)[v * 64];
            }
            if (wave == 0)
#pragma unroll
                for (int v = 0; v < VX; ++v) up[v] = AT(0);
            if (wave + 1 == waves)
#pragma unroll
                for (int v = 0; v < VX; ++v) dn[v] = AT(0);
            const Grid2Step<AT> s = kReread ? step_args(LV - 1) : a.steps[LV - 1];
            Plane &ac = C[SIDE != NONE ? c : 0];
            const Plane *B = L[LV - 1];
            const Plane &aux = L[LV >= 2 ? LV - 2 : 0][c];
            if (LV >= 2 && (s.flags & kG2Aux))
                level<G::AUX>(B[zm], B[c], B[zp], aux, up, dn, s, ac, w);
            else if (s.flags & kG2Unit)
                level<G::UNIT>(B[zm], B[c], B[zp], aux, up, dn, s, ac, w);
            else
                level<G::PLAIN>(B[zm], B[c], B[zp], aux, up, dn, s, ac, w);
        } else {
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int v = 0; v < VX; ++v) w[r][v] = AT(0);
        }
        if constexpr (LV < S) {
            publish(lds, PH & 1, LV, w);
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int v = 0; v < VX; ++v) L[LV][c][r][v] = w[r][v];
        } else if (z >= lo && z < hi) {
            const Global po = plane(a.out, a, z), pa = plane(SIDE == ACC ? a.acc : a.out, a, z);
#pragma unroll
            for (int v = 0; v < VX; ++v) {
#pragma unroll
                for (int r = 0; r < RY; ++r) {
                    if (!((deliver >> (r * VX + v)) & 1)) continue;
                    const unsigned i = off[r] + (unsigned)((v + (VX > 1 ? back : 0)) * (int)sizeof(AT));
                    if constexpr (SIDE == ACC) {
                        at<AT>(pa, i) = C[c][r][v];
                        if (a.out) at<AT>(po, i) = w[r][v];
                    } else if constexpr (SIDE == FIN) {
                        at<AT>(po, i) = C[c][r][v] - w[r][v];
                    } else {
                        at<AT>(po, i) = w[r][v];
                    }
                }
            }
        }
    }

    template <int PH>
    __device__ __forceinline__ void iterate(const G3Args<AT> &a, const AT *side, bool has_side, AT *lds, int t, int z0,
                                            int z1, int last) {
        // The input's plane t was asked for two iterations ago, the side
        // vector's t - 1 one and a bit: the slot it takes was free no earlier.
        pick(a, t < a.gz, L[0][PH]);
        if constexpr (SIDE != NONE) pick(a, has_side, C[(PH - 1) & 3]);
        publish(lds, PH & 1, 0, L[0][PH]);
        advance<PH, 1>(a, lds, t, max(0, z0 - (S - 1)), min(a.gz, z1 + (S - 1)));
        if constexpr (S >= 2) advance<PH, 2>(a, lds, t, max(0, z0 - (S - 2)), min(a.gz, z1 + (S - 2)));
        load(a.in, a, min(t + 2, last), L[0][(PH + 2) & 3]);
        if constexpr (S >= 3) advance<PH, 3>(a, lds, t, z0, z1);
        if constexpr (SIDE != NONE) load(side, a, min(t + 1, last), C[(PH + 1) & 3]);
        __syncthreads();
    }
};

// What bounds it: the issue of the region's operations (14 a point and step
// in FP64, 7 of them FP64), 1.6 to 2.6 times the grid's points with the halos
// of tiles and chunks; the vectors pass through memory once per launch
// instead of once per step. Measured per step, against the best of the other
// chain kernels: FP64 201 x 150 x 97 phi 6.8 us (14.7), p 8.5 us (18.3), 256 x
// 256 x 200 18.2 (33.8) and 36.9 (70.1), 64^3 phi 2.5 (2.7), 30^3 2.1 (3.0);
// FP32 201 x 150 x 97 5.2 (8.1) and 6.5 (11.0), 64^3 2.1 (2.7). Whole-line
// tiles stay the better on 128^3 in FP32: phi 3.4 us against 4.5, p 4.5
// against 5.6.
template <typename AT, int S, int VX, int RY, int SIDE>
__global__ __launch_bounds__((grid3_threads(sizeof(AT), VX, RY))) void k_grid3(G3Args<AT> a) {
    extern __shared__ __align__(16) unsigned char smem[];
    AT *lds = reinterpret_cast<AT *>(smem);
    March3<AT, S, VX, RY, SIDE> m;
    m.lane = threadIdx.x & 63;
    m.waves = (int)(blockDim.x >> 6);
    m.wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int tile = remap_tile(blockIdx.x, a.ntiles, a.remap);
    const int x0 = (tile % a.ntx) * a.tx, y0 = (tile / a.ntx % a.nty) * a.ty, z0 = tile / (a.ntx * a.nty) * a.tz;
    const int z1 = min(z0 + a.tz, a.gz);
    const int x = x0 - a.hx + m.lane * VX, yw = y0 - a.hy + m.wave * RY, xb = min(max(x, 0), a.gx - VX);
    m.back = x - xb;
    m.deliver = 0;
#pragma unroll
    for (int r = 0; r < RY; ++r) m.off[r] = ((unsigned)min(max(yw + r, 0), a.gy - 1) * a.gx + xb) * (unsigned)sizeof(AT);
#pragma unroll
    for (int r = 0; r < RY; ++r)
#pragma unroll
        for (int v = 0; v < VX; ++v) {
            const int px = x + v, py = yw + r;
            m.live[r][v] = px >= 0 && px < a.gx && py >= 0 && py < a.gy;
            if (px >= x0 && px < min(x0 + a.tx, a.gx) && py >= y0 && py < min(y0 + a.ty, a.gy))
                m.deliver |= 1u << (r * VX + v);
        }
#pragma unroll
    for (int d = 0; d < 7; ++d) m.cf[d] = a.coef[d];
    const bool has_side = SIDE == FIN || a.load_acc;
    const AT *side = SIDE == FIN ? a.vfin : (a.load_acc ? a.acc : a.in);
    const int t0 = max(z0 - S, 0), t1 = z1 - 1 + S, last = min(t1, a.gz - 1);
#pragma unroll
    for (int l = 0; l < S; ++l)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int v = 0; v < VX; ++v) m.L[l][k][r][v] = AT(0);
    if constexpr (SIDE != NONE) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int v = 0; v < VX; ++v) m.C[k][r][v] = AT(0);
    }
    m.load(a.in, a, t0, m.L[0][0]);
    m.load(a.in, a, min(t0 + 1, last), m.L[0][1]);
    if constexpr (SIDE != NONE) m.load(side, a, t0, m.C[0]);
    for (int t = t0;;) {
        m.template iterate<0>(a, side, has_side, lds, t, z0, z1, last);
        if (++t > t1) break;
        m.template iterate<1>(a, side, has_side, lds, t, z0, z1, last);
        if (++t > t1) break;
        m.template iterate<2>(a, side, has_side, lds, t, z0, z1, last);
        if (++t > t1) break;
        m.template iterate<3>(a, side, has_side, lds, t, z0, z1, last);
        if (++t > t1) break;
    }
}
template <typename AT, int S, int VX, int RY, int SIDE>
hipError_t g3_launch(const G3Args<AT> &a, const Grid2Shape &s, hipStream_t st) {
    const size_t lds = (size_t)4 * S * s.waves * VX * 64 * sizeof(AT);
    if (lds > 64 * 1024) {  // per device, and cheap next to such a launch
        const hipError_t e = hipFuncSetAttribute((const void *)&k_grid3<AT, S, VX, RY, SIDE>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_grid3<AT, S, VX, RY, SIDE>), dim3((unsigned)a.ntiles), dim3(64 * s.waves), lds, st, a);
    return hipGetLastError();
}

template <typename AT, int S, int VX, int RY>
hipError_t g3_side(const G3Args<AT> &a, const Grid2Shape &s, hipStream_t st) {
    if (a.vfin) return g3_launch<AT, S, VX, RY, FIN>(a, s, st);
    return a.acc ? g3_launch<AT, S, VX, RY, ACC>(a, s, st) : g3_launch<AT, S, VX, RY, NONE>(a, s, st);
}

template <typename AT, int VX, int RY>
hipError_t g3_steps(const G3Args<AT> &a, const Grid2Shape &s, int n, hipStream_t st) {
    return n == 2 ? g3_side<AT, 2, VX, RY>(a, s, st) : g3_side<AT, 3, VX, RY>(a, s, st);
}

template <typename AT>
hipError_t g3_shape(const G3Args<AT> &a, const Grid2Shape &s, int n, hipStream_t st) {
    switch (s.vx * 10 + s.ry) {
        case 12: return g3_steps<AT, 1, 2>(a, s, n, st);
        case 14: return g3_steps<AT, 1, 4>(a, s, n, st);
        case 22: return g3_steps<AT, 2, 2>(a, s, n, st);
    }
    if constexpr (sizeof(AT) == 4)
        if (s.vx == 2 && s.ry == 4) return g3_steps<AT, 2, 4>(a, s, n, st);
    return hipErrorInvalidValue;
}

template <typename AT>
hipError_t g3_run(const Grid3Mat &m, const AT *coef, const Grid2Shape &s, const Grid2Ptrs &p, int remap,
                  hipStream_t st) {
    G3Args<AT> a;
    long tiles = 0;
    if (p.n < 2 || p.n > kGrid3MaxSteps || !grid3_tiles(m, s, p.n, &a.tx, &a.ty, &tiles) || !coef ||
        (p.acc && p.vfin) || (!p.acc && !p.out))
        return hipErrorInvalidValue;
    a.in = (const AT *)p.in;
    a.out = (AT *)p.out;
    a.acc = (AT *)p.acc;
    a.vfin = (const AT *)p.vfin;
    a.coef = coef;
    a.gx = m.gx;
    a.gy = m.gy;
    a.gz = m.gz;
    a.tz = s.tz;
    a.hx = a.tx == m.gx ? 0 : p.n;
    a.hy = a.ty == m.gy ? 0 : p.n;
    a.ntx = (m.gx + a.tx - 1) / a.tx;
    a.nty = (m.gy + a.ty - 1) / a.ty;
    a.ntiles = (int)tiles;
    a.load_acc = p.acc ? p.load_acc : 0;
    a.remap = remap;
    for (int k = 0; k < p.n; ++k) {
        const Grid2Step<double> &u = p.steps[k];
        const bool aux = (u.flags & kG2Aux) != 0;
        if (aux && k == 0) return hipErrorInvalidValue;
        a.steps[k] = Grid2Step<AT>{(AT)u.a0, (AT)u.a1, (AT)u.a2, (AT)u.b0, (AT)u.b1,
                                   u.flags | (u.a1 == 1.0 && !aux ? kG2Unit : 0)};
    }
    return g3_shape<AT>(a, s, p.n, st);
}

}  // namespace

int grid3_max_waves(int prec, int vx, int ry) { return grid3_threads(prec == 0 ? 8 : 4, vx, ry) / 64; }

bool grid3_built(const Grid3Mat &m, int prec, const Grid2Shape &s) {
    if ((prec != 0 && prec != 1) || !m.coef64 || !m.coef32 || m.gx < 2 || (long)m.gx * m.gy >= (1L << 28)) return false;
    if (s.steps < 2 || s.steps > kGrid3MaxSteps || s.waves < 1 || s.waves > grid3_max_waves(prec, s.vx, s.ry)) return false;
    return (s.vx == 1 && (s.ry == 2 || s.ry == 4)) || (s.vx == 2 && (s.ry == 2 || (s.ry == 4 && prec == 1)));
}

bool grid3_tiles(const Grid3Mat &m, const Grid2Shape &s, int n, int *tx, int *ty, long *tiles) {
    if (s.vx < 1 || s.ry < 1 || s.waves < 1 || s.tz < 1 || m.gx < 2 || m.gy < 1 || m.gz < 1) return false;
    const int w = 64 * s.vx, h = s.waves * s.ry;
    *tx = m.gx <= w ? m.gx : w - 2 * n;
    *ty = m.gy <= h ? m.gy : h - 2 * n;
    if (*tx < 1 || *ty < 1) return false;
    *tiles = (long)((m.gx + *tx - 1) / *tx) * ((m.gy + *ty - 1) / *ty) * ((m.gz + s.tz - 1) / s.tz);
    return *tiles < (1L << 31);
}

// A chunk of z planes takes z + 2 n iterations and two of start-up, each as
// long as any other; the chunk height with the shortest sum over the rounds
// of workgroups that the CUs hold at once (eight waves each).
bool grid3_fit(const Grid3Mat &m, Grid2Shape &s) {
    int tx, ty;
    long nxy;
    s.tz = m.gz;
    if (!grid3_tiles(m, s, s.steps, &tx, &ty, &nxy)) return false;
    const long slots = 256L * std::max(1, 8 / s.waves);
    double best = 1e300;
    for (long c = 1; c <= m.gz; ++c) {
        const long z = (m.gz + c - 1) / c, used = (m.gz + z - 1) / z;
        const double t = (double)((nxy * used + slots - 1) / slots) * (double)(z + 2 * s.steps + 2);
        if (t < best) {
            best = t;
            s.tz = (int)z;
        }
    }
    return grid3_tiles(m, s, s.steps, &tx, &ty, &nxy);
}

hipError_t launch_chain_grid3(const Grid3Mat &m, int prec, const Grid2Shape &s, const Grid2Ptrs &p, int remap,
                              hipStream_t st) {
    if (!grid3_built(m, prec, s)) return hipErrorInvalidValue;
    if (prec == 0) return g3_run<double>(m, m.coef64, s, p, remap, st);
    return g3_run<float>(m, m.coef32, s, p, remap, st);
}

}  // namespace ppg
