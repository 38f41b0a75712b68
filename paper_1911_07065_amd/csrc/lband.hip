// Column bands held in LDS: build and product kernels (see lband.h).
#include "lband.h"

#include <algorithm>

#include "devutil.h"

namespace ppg {
namespace {

constexpr int kSlices = kLbRows / 64;

// One window a workgroup, one row a thread: per band a bitonic sort of (127 -
// entries, row), then each slice's width in pairs into sptr.
__global__ __launch_bounds__(kLbRows) void k_lb_sort(int n, const int32_t *rowptr, const int32_t *colind, int nb, int W,
                                                     int nwin, uint16_t *perm, int32_t *sptr, int *bad) {
    __shared__ uint32_t key[kLbRows];
    const int w = blockIdx.x, t = threadIdx.x, row = w * kLbRows + t;
    int cnt[kLbMaxBands];
#pragma unroll
    for (int b = 0; b < kLbMaxBands; ++b) cnt[b] = 0;
    if (row < n)
        for (int e = rowptr[row]; e < rowptr[row + 1]; ++e) {
            const int cb = colind[e] / W;
#pragma unroll
            for (int b = 0; b < kLbMaxBands; ++b) cnt[b] += cb == b ? 1 : 0;
        }
#pragma unroll
    for (int b = 0; b < kLbMaxBands; ++b) {
        if (b >= nb) break;
        if (cnt[b] > kLbMaxEntries) *bad = 1;
        key[t] = (uint32_t)(kLbMaxEntries - min(cnt[b], kLbMaxEntries)) << 9 | (uint32_t)t;
        __syncthreads();
        for (int k = 2; k <= kLbRows; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                const int o = t ^ j;
                const uint32_t a = key[t], c = key[o];
                __syncthreads();
                const bool up = (t & k) == 0, low = t < o;
                key[t] = (low == up) ? min(a, c) : max(a, c);
                __syncthreads();
            }
        const uint32_t v = key[t];
        const long q0 = ((long)b * nwin + w) * kSlices;
        const int len = kLbMaxEntries - (int)(v >> 9);
        perm[(q0 + t / 64) * 64 + t % 64] = (uint16_t)(len << 9 | (v & (kLbRows - 1)));
        if (t % 64 == 0) sptr[q0 + t / 64] = (len + 1) / 2;
        __syncthreads();
    }
}

// sptr[0 .. ns) widths -> exclusive sums, their total in sptr[ns]; one workgroup.
__global__ __launch_bounds__(1024) void k_lb_scan(int ns, int32_t *sptr) {
    __shared__ int32_t sm[1024];
    const int t = threadIdx.x, per = (ns + 1023) / 1024;
    const int i0 = min(ns, t * per), i1 = min(ns, i0 + per);
    int32_t sum = 0;
    for (int i = i0; i < i1; ++i) sum += sptr[i];
    sm[t] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int32_t v = t >= d ? sm[t - d] : 0;
        __syncthreads();
        sm[t] += v;
        __syncthreads();
    }
    int32_t run = sm[t] - sum;
    for (int i = i0; i < i1; ++i) {
        const int32_t w = sptr[i];
        sptr[i] = run;
        run += w;
    }
    if (t == 1023) sptr[ns] = sm[1023];
}

// One wave a slice: each lane walks its row's entries in CSR order.
__global__ __launch_bounds__(256) void k_lb_fill(int n, const int32_t *rowptr, const int32_t *colind, int nb, int W,
                                                 int nwin, const uint16_t *perm, const int32_t *sptr, uint32_t *col,
                                                 int32_t *eperm) {
    const int q = blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= nb * nwin * kSlices) return;
    const int band = q / (nwin * kSlices), w = q / kSlices % nwin;
    const int p0 = sptr[q], width = sptr[q + 1] - p0;
    const int row = w * kLbRows + (perm[(long)q * 64 + lane] & (kLbRows - 1));
    int e = row < n ? rowptr[row] : 0;
    const int e1 = row < n ? rowptr[row + 1] : 0;
    const auto next = [&](uint32_t &c) -> int32_t {
        c = 0;
        while (e < e1) {
            const int cc = colind[e] - band * W;
            ++e;
            if (cc >= 0 && cc < W) {
                c = (uint32_t)cc;
                return e - 1;
            }
        }
        return -1;
    };
    for (int k = 0; k < width; ++k) {
        const long at = (long)(p0 + k) * 64 + lane;
        uint32_t c0, c1;
        eperm[2 * at] = next(c0);
        eperm[2 * at + 1] = next(c1);
        col[at] = c0 | c1 << 16;
    }
}

template <typename VT>
__global__ __launch_bounds__(256) void k_lb_values(long m, const int32_t *eperm, const double *val, VT *out) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i < m) out[i] = eperm[i] >= 0 ? (VT)val[eperm[i]] : VT(0);
}

// The band's part of every row's sum. Workgroup (group, band): its band of the
// input goes to LDS once, then each wave takes slices of the group's windows.
// The first pairs of a wave's next slice are loaded before the current one's
// gathers, and the first slice's before the band is in LDS.
//
// What bounds it: a stream of 6 bytes an entry and the band's copy to LDS. A
// gather from L2 instead is one request an entry at 195 G/s: 250,007 rows x
// 17 entries take 20.5 us a step in BF16 that way, 11.6 us here with the
// launch that adds the bands up (FP32 21.4 and 15.5 us, 130,000 rows 11.4 and
// 8.7 us, 500,000 rows in BF16 27.5 and 22.7 us).
// NP: pairs of a slice loaded before it is used.
template <typename VT, typename XT, int NP>
__global__ __launch_bounds__(1024) void k_lb_product(int n, int W, int nwin, int groups, const int32_t *__restrict__ sptr,
                                                     const uint16_t *__restrict__ perm, const uint32_t *__restrict__ col,
                                                     const VT *__restrict__ val, const XT *__restrict__ in,
                                                     typename Arith<XT>::T *__restrict__ part, int nblocks, int remap) {
    using AT = typename Arith<XT>::T;
    typedef VT V2 __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) unsigned char smem[];
    XT *xs = reinterpret_cast<XT *>(smem);
    const int t = remap_tile(blockIdx.x, nblocks, remap), band = t / groups, g = t - band * groups;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ns = nwin * kSlices;
    const int q0 = (int)((long)ns * g / groups), q1 = (int)((long)ns * (g + 1) / groups);
    const long qb = (long)band * ns;
    const V2 *v2 = reinterpret_cast<const V2 *>(val);
    // slice q: its pairs and this lane's row and length; the first NP pairs
    struct Slice {
        int p, width, pm;
        uint32_t c[NP];
        V2 v[NP];
    };
    auto fetch = [&](int q, Slice &s) {
        s.p = sptr[qb + q];
        s.width = sptr[qb + q + 1] - s.p;
        s.pm = perm[(qb + q) * 64 + lane];
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            // past the slice's end the next slice's pairs (or the padding after
            // the last) are read and dropped
            s.c[k] = col[(long)(s.p + k) * 64 + lane];
            s.v[k] = v2[(long)(s.p + k) * 64 + lane];
        }
    };
    Slice cur, nxt;
    int q = q0 + wave;
    if (q < q1) fetch(q, cur);
    {
        const XT *src = in + (long)band * W;
        const int m = min(W, n - band * W);
        constexpr int E = 16 / (int)sizeof(XT);
        if (((uintptr_t)src & 15) == 0 && m >= E) {
            // all of a thread's loads (at most kLbBytes / 16 KB = 8) before its
            // first store; past the band's end the last word again
            constexpr int NL = kLbBytes / (16 * 1024);
            const int mv = m / E;
            int4 r[NL];
#pragma unroll
            for (int j = 0; j < NL; ++j)
                r[j] = reinterpret_cast<const int4 *>(src)[min((int)threadIdx.x + j * 1024, mv - 1)];
#pragma unroll
            for (int j = 0; j < NL; ++j)  // keeps every load ahead of the stores' tests
                asm volatile("" : "+v"(r[j].x), "+v"(r[j].y), "+v"(r[j].z), "+v"(r[j].w));
#pragma unroll
            for (int j = 0; j < NL; ++j)
                if ((int)threadIdx.x + j * 1024 < mv) reinterpret_cast<int4 *>(xs)[threadIdx.x + j * 1024] = r[j];
            for (int i = mv * E + threadIdx.x; i < m; i += 1024) xs[i] = src[i];
        } else {
            for (int i = threadIdx.x; i < m; i += 1024) xs[i] = src[i];
        }
    }
    __syncthreads();
    for (; q < q1; q += 16) {
        if (q + 16 < q1) fetch(q + 16, nxt);
        const int len = cur.pm >> 9;
        AT s = AT(0);
        auto add = [&](uint32_t c, V2 v, int k) {
            const AT x0 = ldx(xs, (long)(c & 0xffffu)), x1 = ldx(xs, (long)(c >> 16));
            s += 2 * k < len ? (AT)v[0] * x0 : AT(0);
            s += 2 * k + 1 < len ? (AT)v[1] * x1 : AT(0);
        };
#pragma unroll
        for (int k = 0; k < NP; ++k)
            if (cur.width > k) add(cur.c[k], cur.v[k], k);
        for (int k = NP; k < cur.width; k += 2) {
            const long a0 = (long)(cur.p + k) * 64 + lane, a1 = (long)(cur.p + min(k + 1, cur.width - 1)) * 64 + lane;
            const uint32_t c0 = col[a0], c1 = col[a1];
            const V2 w0 = v2[a0], w1 = v2[a1];
            add(c0, w0, k);
            if (k + 1 < cur.width) add(c1, w1, k + 1);
        }
        const int row = q / kSlices * kLbRows + (cur.pm & (kLbRows - 1));
        if (row < n) part[(long)band * n + row] = s;
        cur = nxt;
    }
}

template <typename VT, typename XT, int NP>
hipError_t lb_product_np(const LBand &b, int n, const void *in, int remap, hipStream_t st) {
    using AT = typename Arith<XT>::T;
    const size_t lds = (size_t)b.W * sizeof(XT);
    if (lds > 64 * 1024) {  // per device, and cheap next to such a launch
        const hipError_t e = hipFuncSetAttribute((const void *)&k_lb_product<VT, XT, NP>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    // one workgroup a CU (its LDS): as many groups of slices as make about 256
    const int groups = std::max(1, std::min(256 / b.nb, b.nwin * kSlices)), nblocks = groups * b.nb;
    hipLaunchKernelGGL((k_lb_product<VT, XT, NP>), dim3(nblocks), dim3(1024), lds, st, n, b.W, b.nwin, groups, b.sptr,
                       b.perm, b.col, (const VT *)b.val, (const XT *)in, (AT *)b.part, nblocks, remap);
    return hipGetLastError();
}

// Three pairs ahead when a slice has two or more on average, else two: what
// is loaded past a slice's end is read again with the next one (500,007 rows
// in 8 bands, 1.3 pairs a slice: 22.7 us with two, 26.6 with three; 250,007
// rows in 4 bands, 2.4 pairs: 12.6 and 11.6 us).
template <typename VT, typename XT>
hipError_t lb_product(const LBand &b, int n, const void *in, int remap, hipStream_t st) {
    static_assert(kLbAhead == 3, "the copy is padded for three pairs ahead");
    if (b.pairs >= 2L * b.nb * b.nwin * kSlices) return lb_product_np<VT, XT, 3>(b, n, in, remap, st);
    return lb_product_np<VT, XT, 2>(b, n, in, remap, st);
}

}  // namespace

int lb_bands(int n, size_t elem, int *W) {
    const long cap = std::min<long>(kLbBytes / (long)elem, 65536);
    const long nb = (n + cap - 1) / cap;
    if (nb < 1 || nb > kLbMaxBands) return 0;
    *W = (int)(((n + nb - 1) / nb + 63) / 64 * 64);
    return (int)((n + *W - 1) / *W);
}

hipError_t launch_lb_sort(int n, const int32_t *rowptr, const int32_t *colind, const LBand &b, int *bad,
                          hipStream_t st) {
    hipLaunchKernelGGL(k_lb_sort, dim3(b.nwin), dim3(kLbRows), 0, st, n, rowptr, colind, b.nb, b.W, b.nwin, b.perm,
                       b.sptr, bad);
    hipLaunchKernelGGL(k_lb_scan, dim3(1), dim3(1024), 0, st, b.nb * b.nwin * kSlices, b.sptr);
    return hipGetLastError();
}

hipError_t launch_lb_fill(int n, const int32_t *rowptr, const int32_t *colind, const LBand &b, hipStream_t st) {
    const int ns = b.nb * b.nwin * kSlices;
    hipLaunchKernelGGL(k_lb_fill, dim3((ns + 3) / 4), dim3(256), 0, st, n, rowptr, colind, b.nb, b.W, b.nwin, b.perm,
                       b.sptr, b.col, b.eperm);
    return hipGetLastError();
}

hipError_t launch_lb_values(const LBand &b, bool f64, const double *val, hipStream_t st) {
    const long m = b.pairs * 128;
    if (m == 0) return hipSuccess;
    const dim3 g((unsigned)((m + 255) / 256));
    if (f64)
        hipLaunchKernelGGL(k_lb_values<double>, g, dim3(256), 0, st, m, b.eperm, val, (double *)b.val);
    else
        hipLaunchKernelGGL(k_lb_values<float>, g, dim3(256), 0, st, m, b.eperm, val, (float *)b.val);
    return hipGetLastError();
}

hipError_t launch_lb_product(const LBand &b, int prec, int n, const void *in, int remap, hipStream_t st) {
    if (b.nb < 1 || !b.val) return hipErrorInvalidValue;
    switch (prec) {
        case 0: return lb_product<double, double>(b, n, in, remap, st);
        case 1: return lb_product<float, float>(b, n, in, remap, st);
        case 2: return lb_product<float, uint16_t>(b, n, in, remap, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace ppg
