// Mask predictor kernels for gfx950 (wave64).
//
// All predictor arithmetic is fp64: the block sums of bf16 values are exact
// in fp64, and the statistic, the fit and the scores then agree with an fp64
// reference to rounding level, so the integer outcome (which blocks are kept)
// only depends on the float32 ranking keys.  Every reduction runs in a fixed
// order (no floating-point atomics), so results are bitwise reproducible.
//
// Paper references: block pooling + mass estimate stand in for the sparsity
// map of Eq. 2; the fit solves the normal equations of Eq. 4 with the block
// structure of Appendix B.4; the prediction is the linear extrapolation of
// Section 5.2; the selection implements the ranking and the gated
// block-diagonal support of Section 5.3.
#include "moddit_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace moddit {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxSumRows = 16;   // rows of a map that one work-group sums at most

// f(integral_constant<int, i>) for i = A .. B-1.
template <int A, int B, class Fn>
inline void static_for(Fn&& f) {
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}

inline unsigned cdiv(long a, long b) { return static_cast<unsigned>((a + b - 1) / b); }

__device__ inline double bf16_bits_to_double(uint32_t bits) {
    return static_cast<double>(__uint_as_float(bits << 16));
}

// Fixed-order tree reductions over one 256-thread workgroup.
__device__ double block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    double r = red[0];
    __syncthreads();
    return r;
}

// Exclusive scan over the NT threads of a workgroup in thread order (a
// wave scan, then the wave totals added in wave order: a fixed order).
// wsum: NT / 64 entries of LDS scratch; *total receives the sum.
template <class T, int NT>
__device__ T block_exclusive_scan(T v, T* wsum, T* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    T incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    T base = T(0), all = T(0);
#pragma unroll
    for (int ww = 0; ww < NT / 64; ++ww) {
        if (ww < w) base += wsum[ww];
        all += wsum[ww];
    }
    __syncthreads();   // wsum may be reused by the caller
    *total = all;
    return base + (incl - v);
}

// In-place inclusive prefix sum of a[0 .. len) in LDS over one work-group:
// thread t scans its contiguous segment, the segment totals are scanned in
// thread order, and each segment adds its offset (a fixed order).  Every
// thread of the work-group calls it; a is complete on return.
template <int NT>
__device__ void block_inclusive_prefix(double* a, int len, double* wsum) {
    const int seg = (len + NT - 1) / NT;
    const int b0 = min(len, (int)threadIdx.x * seg), b1 = min(len, b0 + seg);
    double run = 0.0;
    for (int b = b0; b < b1; ++b) {
        run += a[b];
        a[b] = run;
    }
    double total;
    const double off = block_exclusive_scan<double, NT>(run, wsum, &total);
    for (int b = b0; b < b1; ++b) a[b] += off;
    __syncthreads();
}

// ---------------------------------------------------------------------------
// a1: block pooling.  Grid (n, BH, 2): z = 0 pools Q, z = 1 pools K.  The
// block is one contiguous run of rows*D bf16.  Lane l of wave w reads the
// 16-byte chunk l % C (C = D / 8 chunks per row) of rows p*RPP + w*RPW +
// l / C of every pass p; all of a thread's loads (non-temporal) are issued
// before any is used (the whole 32 KB block in flight per work-group), and
// accumulated in fp64.  The rows of a wave are then folded with lane shuffles (xor C, 2C,
// ...), the four waves' sums through LDS in wave order: a fixed summation
// order.  L: tokens pooled (the video tokens); L_stride: tokens per head in
// memory.
// ---------------------------------------------------------------------------
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <int D, int BS>
__global__ __launch_bounds__(kThreads) void pool_kernel(const uint16_t* __restrict__ q,
                                                        const uint16_t* __restrict__ k,
                                                        double* __restrict__ qbar,
                                                        double* __restrict__ kbar, int L,
                                                        int L_stride, int n) {
    constexpr int C = D / 8;               // 16-byte chunks per row
    constexpr int NW = kThreads / 64;      // waves
    constexpr int RPW = 64 / C;            // rows per wave per pass
    constexpr int RPP = NW * RPW;          // rows per pass
    constexpr int NP = BS / RPP;           // passes
    static_assert(BS % RPP == 0, "block rows must fill whole passes");
    __shared__ double part[NW][D];
    const int i = blockIdx.x, bh = blockIdx.y;
    const uint16_t* src = (blockIdx.z == 0 ? q : k) + ((size_t)bh * L_stride + (size_t)i * BS) * D;
    double* dst = (blockIdx.z == 0 ? qbar : kbar) + ((size_t)bh * n + i) * D;
    const int cnt = min(BS, L - i * BS);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, c = lane % C, rs = lane / C;
    uint4 v[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int r = p * RPP + w * RPW + rs;
        // read once and never again: non-temporal loads keep the stream out of the caches
        v[p] = r < cnt ? __builtin_bit_cast(uint4, __builtin_nontemporal_load(
                             reinterpret_cast<const u32x4*>(src + (size_t)r * D + c * 8)))
                       : make_uint4(0, 0, 0, 0);
    }
    double acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t ws[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[2 * e] += bf16_bits_to_double(ws[e] & 0xFFFFu);
            acc[2 * e + 1] += bf16_bits_to_double(ws[e] >> 16);
        }
    }
#pragma unroll
    for (int off = C; off < 64; off <<= 1)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], off);
    if (rs == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) part[w][c * 8 + e] = acc[e];
    }
    __syncthreads();
    if (t < D) {
        double sum = 0.0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) sum += part[ww][t];
        dst[t] = sum / static_cast<double>(cnt);
    }
}

// ---------------------------------------------------------------------------
// a2 (part 1): block logits scale * qbar_i . kbar_j with fp64 matrix
// products (v_mfma_f64_16x16x4_f64): a T x T tile per work-group, T/2 x T/2
// per wave (product tiles of 16 x 16, those past the last block left out),
// channels staged through LDS 16 at a time.  Operand layout of the product
// (16 x 4 times 4 x 16): lane l supplies A[l % 16][l / 16] and B[l / 16]
// [l % 16], and holds D[l / 16 + 4 e][l % 16] in element e of its result.
// T = 64 keeps five waves per SIMD (one group's stores run beside another's
// products); T = 32 where that would leave compute units without work.  24
// heads of 929 blocks, d = 128, predictions back to back: 136 us with 128 x 128
// tiles (two waves per SIMD, whose stores all came at the same time), 118 us
// with 64 x 64 (45 TFLOP/s; an fp64 matrix product of the library runs at 72);
// within a layer step, after the attention, 129-132 us (40-41 TFLOP/s).
// ---------------------------------------------------------------------------
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int D, int T>
__global__ __launch_bounds__(kThreads) void logits_kernel(const double* __restrict__ qbar,
                                                          const double* __restrict__ kbar,
                                                          double* __restrict__ G, int n,
                                                          double scale) {
    constexpr int KC = 16, WT = T / 2, NT = WT / 16;
    static_assert(D % KC == 0 && kThreads == 256, "four waves, 16-channel chunks");
    __shared__ double qs[T][KC + 1];
    __shared__ double ks[T][KC + 1];
    const int bh = blockIdx.z, i0 = blockIdx.y * T, j0 = blockIdx.x * T;
    const double* qb = qbar + (size_t)bh * n * D;
    const double* kb = kbar + (size_t)bh * n * D;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = (w >> 1) * WT, wc = (w & 1) * WT;   // the wave's sub-tile
    const int lm = lane & 15, lk = lane >> 4;
    // product tiles with a row and a column inside the map
    const int nu = (min(WT, n - i0 - wr) + 15) / 16, nv = (min(WT, n - j0 - wc) + 15) / 16;
    f64x4 acc[NT][NT];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int v = 0; v < NT; ++v) acc[u][v] = f64x4{0.0, 0.0, 0.0, 0.0};
    // the next chunk is loaded into registers while this one is multiplied
    constexpr int PT = T * KC / kThreads;   // values of each operand per thread
    double qn[PT], kn[PT];
    auto fetch = [&](int d0) {
#pragma unroll
        for (int x = 0; x < PT; ++x) {
            const int e = threadIdx.x + x * kThreads, r = e / KC, c = e % KC;
            qn[x] = (i0 + r < n) ? qb[(size_t)(i0 + r) * D + d0 + c] : 0.0;
            kn[x] = (j0 + r < n) ? kb[(size_t)(j0 + r) * D + d0 + c] : 0.0;
        }
    };
    fetch(0);
    for (int d0 = 0; d0 < D; d0 += KC) {
#pragma unroll
        for (int x = 0; x < PT; ++x) {
            const int e = threadIdx.x + x * kThreads, r = e / KC, c = e % KC;
            qs[r][c] = qn[x];
            ks[r][c] = kn[x];
        }
        __syncthreads();
        if (d0 + KC < D) fetch(d0 + KC);
#pragma unroll
        for (int kk = 0; kk < KC; kk += 4) {
            double a[NT], b[NT];
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                a[u] = qs[wr + 16 * u + lm][kk + lk];
                b[u] = ks[wc + 16 * u + lm][kk + lk];
            }
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                if (u >= nu) continue;
#pragma unroll
                for (int v = 0; v < NT; ++v)
                    if (v < nv) acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + wr + 16 * u + lk + 4 * e;
            if (i >= n) continue;
#pragma unroll
            for (int v = 0; v < NT; ++v) {
                const int j = j0 + wc + 16 * v + lm;
                if (j < n) G[((size_t)bh * n + i) * n + j] = scale * acc[u][v][e];
            }
        }
}

// The wave's total and maximum of a per-lane double in a fixed order, the
// same bits in every lane: within rows of 16 lanes by DPP (lane pairs, quad
// pairs, then rotations by 4 and 8, after which lane 0 of a row holds its
// row's result), then the four rows' results read from lanes 0, 16, 32, 48.
__device__ inline double dpp_f64(double v, int ctrl_id) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    uint32_t lo = static_cast<uint32_t>(u), hi = static_cast<uint32_t>(u >> 32);
    switch (ctrl_id) {
        case 0: lo = __builtin_amdgcn_mov_dpp((int)lo, 0xB1, 0xF, 0xF, false);
                hi = __builtin_amdgcn_mov_dpp((int)hi, 0xB1, 0xF, 0xF, false); break;   // quad_perm 1,0,3,2
        case 1: lo = __builtin_amdgcn_mov_dpp((int)lo, 0x4E, 0xF, 0xF, false);
                hi = __builtin_amdgcn_mov_dpp((int)hi, 0x4E, 0xF, 0xF, false); break;   // quad_perm 2,3,0,1
        case 2: lo = __builtin_amdgcn_mov_dpp((int)lo, 0x124, 0xF, 0xF, false);
                hi = __builtin_amdgcn_mov_dpp((int)hi, 0x124, 0xF, 0xF, false); break;  // row_ror:4
        default: lo = __builtin_amdgcn_mov_dpp((int)lo, 0x128, 0xF, 0xF, false);
                 hi = __builtin_amdgcn_mov_dpp((int)hi, 0x128, 0xF, 0xF, false); break; // row_ror:8
    }
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

__device__ inline double readlane_f64(double v, int l) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(u), l);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(u >> 32), l);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

__device__ inline double wave_total_f64(double v) {
    v += dpp_f64(v, 0);
    v += dpp_f64(v, 1);
    v += dpp_f64(v, 2);
    v += dpp_f64(v, 3);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

__device__ inline double wave_max_f64(double v) {
    v = fmax(v, dpp_f64(v, 0));
    v = fmax(v, dpp_f64(v, 1));
    v = fmax(v, dpp_f64(v, 2));
    v = fmax(v, dpp_f64(v, 3));
    return fmax(fmax(readlane_f64(v, 0), readlane_f64(v, 16)), fmax(readlane_f64(v, 32), readlane_f64(v, 48)));
}

template <class T>
__device__ inline T wave_inclusive_scan(T v, int lane) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T y = __shfl_up(v, off);
        if (lane >= off) v += y;
    }
    return v;
}

// p / s from s and inv = 1 / s: one correction step, which leaves the
// quotient as the division rounds it but for rare last bits.
__device__ inline double quotient(double p, double s, double inv) {
    const double g = p * inv;
    return fma(fma(-g, s, p), inv, g);
}

// ---------------------------------------------------------------------------
// a2 (part 2) + a3 (sums): a work-group takes R consecutive rows of one
// head's map.  SOFTMAX: each row of logits becomes
//   G(i, j) = |j| exp(l_ij - max_j l) / sum_j |j| exp(...)
// in place; else the map is only read.  Its entries are added into the column
// sums (thread t owns columns t + 256 e, in registers) and the diagonal sums
// (in LDS; consecutive rows shift a diagonal's owner by one thread, and the
// barriers of the row's reductions lie between) of these rows, stored as this
// chunk's part of the right-hand side r = M^T vec(G).  One pass over the map
// instead of three (softmax, diagonals, columns); every sum has a fixed order.
// Bound by the fp64 exponentials and the map's traffic: 24 heads of 929
// blocks (166 MB) 76 us within a layer step (67 us in predictions back to
// back), against 77 + 76 us for a softmax pass and a pass with one thread per
// diagonal or column.
// ---------------------------------------------------------------------------
template <int EPT, bool SOFTMAX>
__global__ __launch_bounds__(kThreads) void map_sums_kernel(double* __restrict__ G, double* __restrict__ part,
                                                            int L, int bs, int n, int R) {
    constexpr int NW = kThreads / 64;
    static_assert(NW == 4, "the wave totals are added as (w0 + w1) + (w2 + w3)");
    __shared__ double dacc[kThreads * EPT + kMaxSumRows];   // diagonal j - i at j - i + i0 + R - 1
    __shared__ double rmax[2][NW], rsum[2][NW];
    const int bh = blockIdx.y, ch = blockIdx.x, nch = gridDim.x;
    const int i0 = ch * R, rows = min(R, n - i0);
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    double* g = G + ((size_t)bh * n + i0) * n;
    for (int a = t; a < n + R - 1; a += kThreads) dacc[a] = 0.0;
    double col[EPT], x[EPT], wgt[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = t + kThreads * e;
        col[e] = 0.0;
        wgt[e] = static_cast<double>(min(bs, L - j * bs));
        x[e] = j < n ? g[j] : -INFINITY;
    }
    for (int r = 0; r < rows; ++r) {
        double nx[EPT];
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int j = t + kThreads * e;
            nx[e] = (r + 1 < rows && j < n) ? g[(size_t)(r + 1) * n + j] : -INFINITY;
        }
        if constexpr (SOFTMAX) {
            double m = x[0];
#pragma unroll
            for (int e = 1; e < EPT; ++e) m = fmax(m, x[e]);
            m = wave_max_f64(m);
            if (lane == 0) rmax[r & 1][w] = m;
            __syncthreads();
            m = fmax(fmax(rmax[r & 1][0], rmax[r & 1][1]), fmax(rmax[r & 1][2], rmax[r & 1][3]));
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                if (t + kThreads * e < n) {
                    x[e] = wgt[e] * exp(x[e] - m);
                    s += x[e];
                }
            }
            s = wave_total_f64(s);
            if (lane == 0) rsum[r & 1][w] = s;
            __syncthreads();
            s = (rsum[r & 1][0] + rsum[r & 1][1]) + (rsum[r & 1][2] + rsum[r & 1][3]);
            const double inv = 1.0 / s;
#pragma unroll
            for (int e = 0; e < EPT; ++e) {
                const int j = t + kThreads * e;
                if (j < n) {
                    x[e] = quotient(x[e], s, inv);
                    g[(size_t)r * n + j] = x[e];
                }
            }
        } else {
            __syncthreads();   // the last row's diagonal sums are complete
        }
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int j = t + kThreads * e;
            if (j < n) {
                col[e] += x[e];
                dacc[j - r + R - 1] += x[e];
            }
            x[e] = nx[e];
        }
    }
    __syncthreads();
    double* out = part + ((size_t)bh * nch + ch) * (2 * n + R - 1);
    for (int a = t; a < n + R - 1; a += kThreads) out[a] = dacc[a];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = t + kThreads * e;
        if (j < n) out[n + R - 1 + j] = col[e];
    }
}

// The chunks' diagonal and column sums added in chunk order, and the sums of
// the frame squares (one work-group per frame, a fixed assignment of entries
// to threads and a fixed-order tree).  Grid (ceil((3n - 1) / 256) + F, BH).
__global__ __launch_bounds__(kThreads) void rhs_kernel(const double* __restrict__ part,
                                                       const double* __restrict__ G,
                                                       const int* __restrict__ reg, double* __restrict__ r,
                                                       int n, int F, int nch, int R) {
    __shared__ double red[kThreads];
    const int bh = blockIdx.y, nb = gridDim.x - F;
    double* rr = r + (size_t)bh * (3 * n - 1 + F);
    if ((int)blockIdx.x >= nb) {
        const int f = blockIdx.x - nb;
        const int lo = reg[2 * f], hi = reg[2 * f + 1], sz = hi - lo + 1;
        const double* g = G + (size_t)bh * n * n;
        double s = 0.0;
        for (int e = threadIdx.x; e < sz * sz; e += kThreads) s += g[(size_t)(lo + e / sz) * n + lo + e % sz];
        s = block_sum(s, red);
        if (threadIdx.x == 0) rr[3 * n - 1 + f] = s;
        return;
    }
    const int o = blockIdx.x * kThreads + threadIdx.x;
    if (o >= 3 * n - 1) return;
    const int stride = 2 * n + R - 1;
    const double* pp = part + (size_t)bh * nch * stride;
    int ca = 0, cb = nch - 1, at = n + R - 1 + (o - (2 * n - 1)), step = stride;   // a column
    if (o < 2 * n - 1) {
        // diagonal dl lies in chunk c at dl + c R + R - 1, if
        // that is in [0, n + R - 2]
        const int dl = o - (n - 1);
        ca = max(0, -dl / R);
        cb = min(nch - 1, (n - 1 - dl) / R);
        at = dl + R - 1;
        step = stride + R;
    }
    double s = 0.0;
#pragma unroll 8
    for (int c = ca; c <= cb; ++c) s += pp[(ptrdiff_t)c * step + at];
    rr[o] = s;
}

// ---------------------------------------------------------------------------
// a3 (solve).  The normal matrix N = M^T M has a diagonal C^T C block
// (Appendix B.4).  Fixing the gauge by dropping the last vertical column,
// the unknowns split into c (2n-1) and u = [d_0..d_{n-2}, e] (q = n-1+F):
//   [Dc  W ] [c]   [r_C]          S = Y - W^T Dc^{-1} W   (host, inverted)
//   [W^T Y ] [u] = [r_U],         u = S^{-1} (r_U - W^T Dc^{-1} r_C)
//                                 c = Dc^{-1} (r_C - W u)
// with Dc = diag(n - |delta|), W[delta, j] = 1 iff column j crosses
// diagonal delta, W[delta, f] = max(0, |R_f| - |delta|).  The result is
// moved to the minimum-norm gauge by removing its component along
// z = [1, -1, 0].
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void solve_pre_kernel(const double* __restrict__ r,
                                                             const int* __restrict__ reg,
                                                             double* __restrict__ bU, int n,
                                                             int F) {
    extern __shared__ double y[];   // 2n - 1: Dc^{-1} r_C, then its inclusive prefix
    __shared__ double wsum[kThreads / 64];
    const int bh = blockIdx.y;      // x: a chunk of kThreads outputs
    const int p = 3 * n - 1 + F, q = n - 1 + F;
    const double* rr = r + (size_t)bh * p;
    for (int a = threadIdx.x; a < 2 * n - 1; a += kThreads)
        y[a] = rr[a] / static_cast<double>(n - abs(a - (n - 1)));
    __syncthreads();
    const int j = blockIdx.x * kThreads + threadIdx.x;
    // frame rows of W^T: weighted sums of the diagonals a frame square spans
    double s = 0.0;
    if (j >= n - 1 && j < q) {
        const int f = j - (n - 1);
        const int sz = reg[2 * f + 1] - reg[2 * f] + 1;
        for (int dl = -(sz - 1); dl <= sz - 1; ++dl)
            s += static_cast<double>(sz - abs(dl)) * y[dl + n - 1];
    }
    __syncthreads();
    // column rows of W^T: the n diagonals column j crosses, y[j .. j + n - 1],
    // as a difference of the prefix sums
    block_inclusive_prefix<kThreads>(y, 2 * n - 1, wsum);
    if (j < n - 1) s = y[j + n - 1] - (j > 0 ? y[j - 1] : 0.0);
    if (j < q) bU[(size_t)bh * q + j] = (j < n - 1 ? rr[2 * n - 1 + j] : rr[3 * n - 1 + (j - (n - 1))]) - s;
}

// u[h] = S^{-1} bU[h] for all heads, split over kSolveSplit fixed chunks of
// k and the four waves of a work-group: part[c][h][j] = sum over k in chunk c
// of S^{-1}[k][j] bU[h][k] (S^{-1} symmetric, read row-wise: a wave's lanes
// read 64 consecutive columns; each wave a quarter of the chunk, ascending,
// the quarters added in order).  The post kernel adds the chunks in order, so
// the result does not depend on the launch.  Grid: (column chunks of 64,
// kSolveSplit).  Bound by the latency of S^{-1} (7 MB at n = 929, shared by
// every head), so a wave loads 16 rows at once and reuses them for 8 heads.
__global__ __launch_bounds__(kThreads) void solve_gemv_kernel(const double* __restrict__ Sinv,
                                                              const double* __restrict__ bU,
                                                              double* __restrict__ part, int q,
                                                              int BH) {
    constexpr int HW = 8, KB = 16, NW = kThreads / 64;
    __shared__ double bs[NW][KB][HW];        // a wave's right-hand sides, 16 k at a time
    __shared__ double red[NW][HW][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane;
    const int c = blockIdx.y;
    const int kc = (q + kSolveSplit - 1) / kSolveSplit;
    const int k0 = min(q, c * kc), k1 = min(q, k0 + kc), kw = (k1 - k0 + NW - 1) / NW;
    const int ka = min(k1, k0 + w * kw), kz = min(k1, ka + kw);
    const double* col = Sinv + min(j, q - 1);
    for (int h0 = 0; h0 < BH; h0 += HW) {
        double acc[HW];
#pragma unroll
        for (int hh = 0; hh < HW; ++hh) acc[hh] = 0.0;
        for (int kb = ka; kb < kz; kb += KB) {
            double a[KB];
#pragma unroll
            for (int kk = 0; kk < KB; ++kk) a[kk] = col[(size_t)min(kb + kk, kz - 1) * q];
            // (the wave's LDS operations run in order: the previous pass's
            // reads are done before these writes)
#pragma unroll
            for (int x = 0; x < KB * HW / 64; ++x) {
                const int e = lane + 64 * x, hh = e / KB, kk = e % KB;
                bs[w][kk][hh] = (kb + kk < kz && h0 + hh < BH) ? bU[(size_t)(h0 + hh) * q + kb + kk] : 0.0;
            }
#pragma unroll
            for (int kk = 0; kk < KB; ++kk)
#pragma unroll
                for (int hh = 0; hh < HW; ++hh) acc[hh] = fma(a[kk], bs[w][kk][hh], acc[hh]);
        }
#pragma unroll
        for (int hh = 0; hh < HW; ++hh) red[w][hh][lane] = acc[hh];
        __syncthreads();
#pragma unroll
        for (int x = 0; x < HW / NW; ++x) {
            const int hh = w + NW * x;
            if (j < q && h0 + hh < BH)
                part[((size_t)c * BH + h0 + hh) * q + j] =
                    ((red[0][hh][lane] + red[1][hh][lane]) + red[2][hh][lane]) + red[3][hh][lane];
        }
        __syncthreads();   // red may be rewritten
    }
}

// c = Dc^{-1} (r_C - W u), then the minimum-norm gauge: the component of X
// along z = [1, -1, 0] removed.  One work-group of 1024 threads per head;
// every entry of X that a thread corrects, it wrote itself.
constexpr int kPostThreads = 1024;

__global__ __launch_bounds__(kPostThreads) void solve_post_kernel(const double* __restrict__ r,
                                                                  const double* __restrict__ u,
                                                                  const int* __restrict__ reg,
                                                                  double* __restrict__ X, int n,
                                                                  int F, int BH) {
    extern __shared__ double us[];   // q: u, then the prefix of its first n - 1 entries; then F frame sizes
    __shared__ double wsum[kPostThreads / 64];
    __shared__ int szmax;
    const int bh = blockIdx.x, t = threadIdx.x;
    const int p = 3 * n - 1 + F, q = n - 1 + F;
    int* sz = reinterpret_cast<int*>(us + q);
    if (t == 0) szmax = 0;
    __syncthreads();
    for (int f = t; f < F; f += kPostThreads) {
        sz[f] = reg[2 * f + 1] - reg[2 * f] + 1;
        atomicMax(&szmax, sz[f]);
    }
    const double* rr = r + (size_t)bh * p;
    double* x = X + (size_t)bh * p;
    double net = 0.0;   // sum(c) - sum(d) of this thread's entries
    // u = sum of the k-chunk partial products, in chunk order; the d and e
    // parts of X are u itself (d_{n-1}, the gauge column dropped, is 0)
    for (int a = t; a < q; a += kPostThreads) {
        double v = 0.0;
#pragma unroll
        for (int c = 0; c < kSolveSplit; ++c) v += u[((size_t)c * BH + bh) * q + a];
        us[a] = v;
        if (a < n - 1) net -= v;
        else x[3 * n - 1 + (a - (n - 1))] = v;
    }
    __syncthreads();
    // the d part, before the prefix takes its place
    for (int a = t; a < n; a += kPostThreads) x[2 * n - 1 + a] = a < n - 1 ? us[a] : 0.0;
    __syncthreads();
    block_inclusive_prefix<kPostThreads>(us, n - 1, wsum);
    // c: the columns crossing diagonal dl are a window of d (a difference of
    // the prefix sums), the frames' weights max(0, |R_f| - |dl|) multiply e
    for (int a = t; a < 2 * n - 1; a += kPostThreads) {
        const int dl = a - (n - 1);
        const int j0 = max(0, dl), j1 = min(n - 2, dl + n - 1);
        double s = j1 >= j0 ? us[j1] - (j0 > 0 ? us[j0 - 1] : 0.0) : 0.0;
        if (abs(dl) < szmax) {   // only diagonals shorter than a frame square's side meet one
            for (int f = 0; f < F; ++f) {
                const int w = sz[f] - abs(dl);
                if (w > 0) s += static_cast<double>(w) * us[n - 1 + f];
            }
        }
        const double cv = (rr[a] - s) / static_cast<double>(n - abs(dl));
        x[a] = cv;
        net += cv;
    }
    double total;
    (void)block_exclusive_scan<double, kPostThreads>(net, wsum, &total);
    const double alpha = total / static_cast<double>(3 * n - 1);
    for (int a = t; a < 2 * n - 1; a += kPostThreads) x[a] -= alpha;
    for (int j = t; j < n; j += kPostThreads) x[2 * n - 1 + j] += alpha;
}

// ---------------------------------------------------------------------------
// a2 (part 2) + a3 for short maps (n <= NC, F <= NC): one work-group per head
// holds the map in LDS and goes from the logits (SOFTMAX) or the stored map to
// X in one launch.  The steps are those of map_sums_kernel, rhs_kernel and the
// solve kernels.  A fit of so few blocks is a chain of launches and of
// latencies within them, not work: 8 heads of 64 blocks took 55 us in nine launches, 18 in
// two (logits and this one).
// ---------------------------------------------------------------------------
constexpr int kFitThreads = 1024;

template <int NC, bool SOFTMAX>
__global__ __launch_bounds__(kFitThreads) void fit_small_kernel(double* __restrict__ G, const int* __restrict__ reg,
                                                                const double* __restrict__ Sinv,
                                                                double* __restrict__ X, int L, int bs, int n,
                                                                int F) {
    constexpr int NW = kFitThreads / 64, EW = NC / 64;
    constexpr int SPL = kFitThreads / (4 * NC);     // row ranges of a diagonal's or column's sum
    constexpr int KSPL = kFitThreads / (2 * NC);    // k ranges of the product with S^{-1}
    __shared__ double g[NC][NC + 1];
    __shared__ double rr[4 * NC], y[2 * NC], py[2 * NC], bu[2 * NC], uu[2 * NC], pu[NC];
    __shared__ double part[kFitThreads];
    __shared__ double wsum[NW];
    __shared__ int sz[NC];
    __shared__ int szmax;
    const int bh = blockIdx.x, t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m = 3 * n - 1, q = n - 1 + F;
    double* gg = G + (size_t)bh * n * n;
    if (t == 0) szmax = 0;
    // the map: a wave per row
    for (int i = w; i < n; i += NW) {
        double x[EW];
        double mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < EW; ++e) {
            const int j = lane + 64 * e;
            x[e] = j < n ? gg[(size_t)i * n + j] : -INFINITY;
            mx = fmax(mx, x[e]);
        }
        if constexpr (SOFTMAX) {
            mx = wave_max_f64(mx);
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                const int j = lane + 64 * e;
                if (j < n) {
                    x[e] = static_cast<double>(min(bs, L - j * bs)) * exp(x[e] - mx);
                    s += x[e];
                }
            }
            s = wave_total_f64(s);
            const double inv = 1.0 / s;
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                const int j = lane + 64 * e;
                x[e] = quotient(x[e], s, inv);
                if (j < n) gg[(size_t)i * n + j] = x[e];
            }
        }
#pragma unroll
        for (int e = 0; e < EW; ++e)
            if (lane + 64 * e < n) g[i][lane + 64 * e] = x[e];
    }
    __syncthreads();
    // sums: diagonals and columns over SPL row ranges, frame squares by wave
    for (int f = t; f < F; f += kFitThreads) {
        sz[f] = reg[2 * f + 1] - reg[2 * f] + 1;
        atomicMax(&szmax, sz[f]);
    }
    {
        const int o = t % (4 * NC), c = t / (4 * NC);
        const int r0 = c * n / SPL, r1 = (c + 1) * n / SPL;
        double s = 0.0;
        if (o < 2 * n - 1) {
            const int dl = o - (n - 1);
            for (int i = max(r0, -dl); i < min(r1, n - dl); ++i) s += g[i][i + dl];
        } else if (o < m) {
            for (int i = r0; i < r1; ++i) s += g[i][o - (2 * n - 1)];
        }
        part[t] = s;
    }
    for (int f = w; f < F; f += NW) {
        const int lo = reg[2 * f], side = reg[2 * f + 1] - lo + 1;
        double s = 0.0;
        for (int e = lane; e < side * side; e += 64) s += g[lo + e / side][lo + e % side];
        s = wave_total_f64(s);
        if (lane == 0) rr[m + f] = s;
    }
    __syncthreads();
    if (t < m) {
        double s = part[t];
#pragma unroll
        for (int c = 1; c < SPL; ++c) s += part[c * 4 * NC + t];
        rr[t] = s;
        if (t < 2 * n - 1) y[t] = s / static_cast<double>(n - abs(t - (n - 1)));
    }
    __syncthreads();
    // b_U = r_U - W^T y: prefix sums of y for the columns, a wave per frame
    if (w == NW - 1) {
        constexpr int S = 2 * NC / 64;
        double run = 0.0, v[S];
#pragma unroll
        for (int e = 0; e < S; ++e) {
            const int a = S * lane + e;
            run += a < 2 * n - 1 ? y[a] : 0.0;
            v[e] = run;
        }
        const double off = wave_inclusive_scan(run, lane) - run;
#pragma unroll
        for (int e = 0; e < S; ++e) py[S * lane + e] = v[e] + off;
    }
    for (int f = w; f < F; f += NW) {
        const int side = sz[f];
        double s = 0.0;
        for (int e = lane; e < 2 * side - 1; e += 64) {
            const int dl = e - (side - 1);
            s += static_cast<double>(side - abs(dl)) * y[dl + n - 1];
        }
        s = wave_total_f64(s);
        if (lane == 0) bu[n - 1 + f] = rr[m + f] - s;
    }
    __syncthreads();
    if (t < n - 1) bu[t] = rr[2 * n - 1 + t] - (py[t + n - 1] - (t > 0 ? py[t - 1] : 0.0));
    __syncthreads();
    // u = S^{-1} b_U over KSPL ranges of k
    {
        const int j = t % (2 * NC), c = t / (2 * NC);
        const int k0 = c * q / KSPL, k1 = (c + 1) * q / KSPL;
        double s = 0.0;
        if (j < q) {
#pragma unroll 8
            for (int k = k0; k < k1; ++k) s = fma(Sinv[(size_t)k * q + j], bu[k], s);
        }
        part[t] = s;
    }
    __syncthreads();
    if (t < q) {
        double s = part[t];
#pragma unroll
        for (int c = 1; c < KSPL; ++c) s += part[c * 2 * NC + t];
        uu[t] = s;
    }
    __syncthreads();
    if (w == 0) {
        double run = 0.0, v[EW];
#pragma unroll
        for (int e = 0; e < EW; ++e) {
            const int a = EW * lane + e;
            run += a < n - 1 ? uu[a] : 0.0;
            v[e] = run;
        }
        const double off = wave_inclusive_scan(run, lane) - run;
#pragma unroll
        for (int e = 0; e < EW; ++e) pu[EW * lane + e] = v[e] + off;
    }
    __syncthreads();
    // c = Dc^{-1} (r_C - W u), the gauge, and X
    double v = 0.0, net = 0.0;
    if (t < 2 * n - 1) {
        const int dl = t - (n - 1);
        const int j0 = max(0, dl), j1 = min(n - 2, dl + n - 1);
        double s = j1 >= j0 ? pu[j1] - (j0 > 0 ? pu[j0 - 1] : 0.0) : 0.0;
        if (abs(dl) < szmax) {
            for (int f = 0; f < F; ++f) {
                const int side = sz[f] - abs(dl);
                if (side > 0) s += static_cast<double>(side) * uu[n - 1 + f];
            }
        }
        v = (rr[t] - s) / static_cast<double>(n - abs(dl));
        net = v;
    } else if (t < m) {
        const int j = t - (2 * n - 1);
        v = j < n - 1 ? uu[j] : 0.0;   // d_{n-1}: the gauge column dropped
        net = -v;
    }
    net = wave_total_f64(net);
    if (lane == 0) wsum[w] = net;
    __syncthreads();
    double total = 0.0;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) total += wsum[ww];
    const double alpha = total / static_cast<double>(m);
    double* x = X + (size_t)bh * (m + F);
    if (t < m) x[t] = t < 2 * n - 1 ? v - alpha : v + alpha;
    else if (t < m + F) x[t] = uu[n - 1 + (t - m)];
}

// ---------------------------------------------------------------------------
// Gate: on iff min over the anchors of the frame-averaged e exceeds tau_e.
// ---------------------------------------------------------------------------
__global__ void gate_kernel(const double* __restrict__ Xa, const double* __restrict__ Xb,
                            int32_t* __restrict__ gate, int BH, int n, int F, double tau_e) {
    const int bh = blockIdx.x * blockDim.x + threadIdx.x;
    if (bh >= BH) return;
    const int p = 3 * n - 1 + F;
    double ea = 0.0, eb = 0.0;
    for (int f = 0; f < F; ++f) {
        ea += Xa[(size_t)bh * p + 3 * n - 1 + f];
        eb += Xb[(size_t)bh * p + 3 * n - 1 + f];
    }
    ea /= F;
    eb /= F;
    gate[bh] = fmin(ea, eb) > tau_e ? 1 : 0;
}

// ---------------------------------------------------------------------------
// a4 + a5: extrapolation and per-row selection in one launch.
//
// A work-group of four waves serves consecutive query rows of one head.  It
// extrapolates the diagonals and columns these rows meet (X2 + (X2 - X1) w,
// Section 5.2; n + rows - 1 and n values) and writes its share of the
// prediction.  Up to 2304 blocks each wave then selects rpw rows; beyond, the
// four waves share a row (SHARED), since a wave's 37 to 64 keys per lane leave
// one or two waves per SIMD and all of a step's instructions in one chain.
//
//   sigma_j = n (c~[j-i] + d~[j]) in fp64, rounded to float: the ranking key.
//   The non-forced blocks are ranked by (sigma desc, j asc).  TOPK keeps the
//   first max(0, k - |forced|) of them; MASS keeps the shortest prefix whose
//   positive key mass, added to the forced blocks' mass, reaches tau of the
//   row total (fp64 sums; at least one block).  The kept set is compacted in
//   ascending j.
// Every free block j holds the order bits of its key (vb, 0 for forced blocks
// and padding; block first + lane + 64 e in element e, first the wave's).  The
// kept free blocks are those whose bits exceed a boundary p, plus the first r
// in ascending j of those whose bits equal p.  Both budgets ask for the largest
// threshold at or above which the keys' count (TOPK) or mass (MASS, summed in
// one fixed order) still reaches the target; that predicate only changes at
// keys, so any search finds the same set.  A step costs EW compares with a
// scalar count each (MASS: also EW fp64 additions) and some twenty scalar
// instructions, so few steps are what counts: the search starts at the boundary
// of the row before (neighbouring rows shift the diagonals by one), gallops
// until it has the boundary between two thresholds, halves their distance in
// order bits, and ends once one key lies between them: 10-12 steps for a
// first row, 4-6 for the next ones (interpolating between the counts takes as
// many).  Up to three keys per lane the TOPK boundary is built bit by bit
// instead: 32 steps of a few instructions (TOPK, 25%, 300 heads of 64 blocks
// 11.4 us, 17.7 galloping; 256 of 128 22.8, 28.5; 256 of 190 41.3, 43.5; at
// four keys, 60 of 256 at 5%, 19.4, 15.8).  The ballots that count also place
// the kept blocks, so the stores of a wave are contiguous.
// The lane's block number is made opaque once per row: the lane masks of the
// range and forced tests, kept across rows, spilled scalar registers from 448
// (MASS) and 640 (TOPK) blocks on.
// With the extrapolation: TOPK, 40 heads of 591 blocks 80 -> 41 us; MASS, 24
// heads of 929 blocks 139 -> 71 us; bound by vector issue.  SHARED, 8 heads of
// 2600: TOPK 290 -> 147, MASS 485 -> 259 us (a wave per row: 137 and 273); one
// head of 4096: TOPK 71 -> 60, MASS 113 -> 105 us (82 and 147).
//
// With a text segment after the video (token-type-aware masking) n counts
// the video blocks, the lists have ldn >= n entries per row, the block tb0
// shared by the video and the text (tb0 < n) is forced, and every row keeps
// the text blocks n .. ldn-1 after its video selection; the rows of the text
// blocks (tb0 .. ldn-1, the last work-groups) keep every block.  tb0 >= ldn:
// none.
// ---------------------------------------------------------------------------
__device__ inline double extrapolated(const double* X1, const double* X2, double w, size_t a) {
    const double x2 = X2[a], x1 = X1[a];
    return x2 + (x2 - x1) * w;
}

__device__ inline uint32_t order_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ inline float order_bits_to_float(uint32_t k) {
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// Lanes below this one in a 64-lane mask.
__device__ inline int mask_rank(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A row of a text block: every block kept.
__device__ inline void keep_all(int32_t* __restrict__ kv_idx, int32_t* __restrict__ kv_cnt, size_t orow, int ldn) {
    int32_t* out = kv_idx + orow * ldn;
    for (int j = threadIdx.x; j < ldn; j += kThreads) out[j] = j;
    if (threadIdx.x == 0) kv_cnt[orow] = ldn;
}

constexpr int kWavesPerGroup = kThreads / 64;
constexpr int kMaxRowsPerWave = 2;

// The rows of a selection launch: work-groups 0 .. chunks-1 of a head take
// 4 rpw video rows each, the others one text row.
struct RowGrid {
    int rpw, chunks;
    unsigned groups;
};

RowGrid row_grid(int BH, int n, int ldn, int tb0) {
    // One row per wave until that fills the chip's 1024 SIMDs eight deep;
    // beyond, two, the second starting from the first one's boundary (40 heads
    // of 591 blocks, TOPK 25%: 47 us with one, 41 with two, 41 with four, 45
    // with eight; 24 of 929, MASS: 96, 79, 79 and 85 us with spilled masks, 71
    // and 72 us with two and four without).
    const long rows = (long)BH * n;
    const int rpw = (int)std::max<long>(1, std::min<long>(kMaxRowsPerWave, rows / 4096));
    const int chunks = (n + kWavesPerGroup * rpw - 1) / (kWavesPerGroup * rpw);
    return RowGrid{rpw, chunks, (unsigned)(chunks + std::max(0, ldn - tb0))};
}

constexpr int kWideBlocks = 2304;      // longest row that one wave selects
constexpr int kMaxSharedRows = 4;      // rows of a work-group whose waves share them

// rpw: rows per wave, or (SHARED) per work-group.
template <int EW, bool MASS, bool SHARED>
__global__ __launch_bounds__(kThreads) void select_rows_kernel(
    const double* __restrict__ X1, const double* __restrict__ X2, double w, double* __restrict__ pred,
    const int32_t* __restrict__ gate, const int* __restrict__ row_lo, const int* __restrict__ row_hi, int topk,
    double tau, int32_t* __restrict__ kv_idx, int32_t* __restrict__ kv_cnt, int n, int F, int ldn, int tb0,
    int rpw, int chunks) {
    constexpr int NW = kWavesPerGroup, WPR = SHARED ? NW : 1;                       // waves per row
    constexpr bool BY_BITS = !MASS && !SHARED && EW <= 3;
    __shared__ double cs[64 * EW * WPR + (SHARED ? kMaxSharedRows : NW * kMaxRowsPerWave)];   // diagonals c0 ..
    __shared__ double ds[SHARED ? 1 : 64 * EW];                                     // columns
    __shared__ int xi[2][NW];       // SHARED: the waves' parts of a count and of a mass,
    __shared__ double xd[2][NW];    // two sets in turn (one barrier per exchange)
    const int bh = blockIdx.y;
    if ((int)blockIdx.x >= chunks) {
        keep_all(kv_idx, kv_cnt, (size_t)bh * ldn + tb0 + (blockIdx.x - chunks), ldn);
        return;
    }
    const int m = 3 * n - 1;
    const size_t xo = (size_t)bh * (m + F);
    const int rows = SHARED ? rpw : NW * rpw;
    const int i0 = blockIdx.x * rows;
    const int i1 = min(n, i0 + rows);                    // rows [i0, i1)
    const int c0 = n - i1;                               // diagonal index of (i1 - 1, 0)
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int jw = (SHARED ? wv * 64 * EW : 0) + lane;   // this lane's first block
    for (int a = threadIdx.x; a < n + (i1 - i0) - 1; a += kThreads) cs[a] = extrapolated(X1, X2, w, xo + c0 + a);
    double dr[SHARED ? EW : 1];     // SHARED: the lane's columns stay in registers, which halves the LDS
    if constexpr (SHARED) {
#pragma unroll
        for (int e = 0; e < EW; ++e) dr[e] = extrapolated(X1, X2, w, xo + 2 * n - 1 + min(jw + 64 * e, n - 1));
    } else {
        for (int a = threadIdx.x; a < n; a += kThreads) ds[a] = extrapolated(X1, X2, w, xo + 2 * n - 1 + a);
    }
    {
        const int per = (m + chunks - 1) / chunks, a1 = min(m, ((int)blockIdx.x + 1) * per);
        for (int a = blockIdx.x * per + threadIdx.x; a < a1; a += kThreads)
            pred[(size_t)bh * m + a] = extrapolated(X1, X2, w, xo + a);
    }
    __syncthreads();
    const bool g = gate[bh] != 0;
    int par = 0;
    // SHARED: a wave's count and mass summed over the waves, in wave order
    auto exchange = [&](int& c, double& s) {
        if constexpr (SHARED) {
            if (lane == 0) {
                xi[par][wv] = c;
                if constexpr (MASS) xd[par][wv] = s;
            }
            __syncthreads();
            c = 0;
            s = 0.0;
#pragma unroll
            for (int x = 0; x < NW; ++x) {
                c += xi[par][x];
                if constexpr (MASS) s += xd[par][x];
            }
            par ^= 1;
        }
    };
    // SHARED: the counts of the waves before this one, and of all
    auto before = [&](int c, int& all) {
        if (lane == 0) xi[par][wv] = c;
        __syncthreads();
        int pre = 0;
        all = 0;
#pragma unroll
        for (int x = 0; x < NW; ++x) {
            pre += x < wv ? xi[par][x] : 0;
            all += xi[par][x];
        }
        par ^= 1;
        return pre;
    };
    uint32_t guess = 0xBF800000u;    // 1.0: the score of every block of a uniform map
    uint32_t stride = 1u << 23;      // first gallop step: a factor of two
    for (int rr = 0; rr < rpw; ++rr) {
        const int i = i0 + (SHARED ? 0 : wv * rpw) + rr;
        if (i >= min(i1, tb0)) break;
        int jl = jw;
        asm volatile("" : "+v"(jl));    // no lane mask is kept from one row to the next
        const int flo = row_lo[i], fhi = row_hi[i];
        // forced: the frame blocks of i (gate on) and the block shared by the
        // video and the text segment (tb0 < n), which is a text block
        const bool tb_in_frames = g && tb0 >= flo && tb0 <= fhi;
        const int nf = (g ? (fhi - flo + 1) : 0) + ((tb0 < n && !tb_in_frames) ? 1 : 0);
        const int n_free = n - nf;
        int f0 = flo, f1 = g ? fhi - flo + 1 : 0, f2 = tb0 < n ? tb0 : -1;
        auto is_forced = [&](int j) { return (unsigned)(j - f0) < (unsigned)f1 || j == f2; };

        double forced_mass = 0.0;
        uint32_t vb[EW];
        float ms[SHARED ? 1 : EW];    // positive mass of a free key
#pragma unroll
        for (int e = 0; e < EW; ++e) {
            const int j = jl + 64 * e;
            vb[e] = 0;
            if constexpr (!SHARED) ms[e] = 0.0f;
            if (j < n) {
                double dj;
                if constexpr (SHARED) dj = dr[e];
                else dj = ds[j];
                const double sv = static_cast<double>(n) * (cs[j + (i1 - 1 - i)] + dj);
                const float kf = static_cast<float>(sv);
                if (is_forced(j)) {
                    if constexpr (MASS) forced_mass += fmax(static_cast<double>(kf), 0.0);
                } else {
                    vb[e] = order_bits(kf);
                    if constexpr (!SHARED) ms[e] = fmaxf(kf, 0.0f);
                }
            }
        }
        // the free keys with bits >= th (th >= 1), and (MASS) their mass, in
        // one pass so that no compare's mask outlives its element
        auto at_least = [&](uint32_t th, double& mass) {
            int c = 0;
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                if constexpr (MASS && SHARED) asm volatile("" : "+v"(vb[e]));   // (the mass is not kept beside the bits)
                const bool ge = vb[e] >= th;
                c += __popcll(__ballot(ge));
                if constexpr (MASS) {
                    float me;    // positive keys have the sign bit set in their order bits
                    if constexpr (SHARED) me = fmaxf(__uint_as_float(vb[e] ^ 0x80000000u), 0.0f);
                    else me = ms[e];
                    s += static_cast<double>(ge ? me : 0.0f);
                }
            }
            if constexpr (MASS) s = wave_total_f64(s);
            exchange(c, s);
            mass = s;
            return c;
        };

        uint32_t p = 0;      // boundary bits
        int r = 0;           // keys kept at the boundary, in ascending j
        int keep = -1;       // free keys kept when all or none are
        double fm = 0.0, target = 0.0, mass = 0.0;
        if constexpr (MASS) {
            fm = wave_total_f64(forced_mass);
            int none = 0;
            exchange(none, fm);
            (void)at_least(1u, mass);
            const double total = fm + (n_free > 0 ? mass : 0.0);
            target = tau * total;
            if (fm >= target)
                keep = min(n_free, nf > 0 ? 0 : 1);
            else if (total < target)
                keep = n_free;
        } else {
            keep = min(n_free, max(0, topk - nf));
        }
        if (keep == 0) {
            p = 0xFFFFFFFFu;
        } else if (keep >= n_free) {
            p = 0;
        } else if constexpr (BY_BITS) {
            // the largest p with at least keep free keys at or above it
#pragma unroll
            for (int b = 31; b >= 0; --b) {
                const uint32_t th = p | (1u << b);
                if (at_least(th, mass) >= keep) p = th;
            }
            r = keep - (p < 0xFFFFFFFFu ? at_least(p + 1, mass) : 0);
        } else {
            // lo reaches the target (with c_lo keys), hi does not (c_hi); a
            // bound not yet evaluated has the largest count possible.  By
            // mass the boundary key is positive, so its sign bit is set.
            const bool by_mass = MASS && keep < 0;
            uint32_t lo = by_mass ? 0x80000000u : 1u, hi = 0xFFFFFFFFu;
            int c_lo = n_free, c_hi = 0;
            bool have_lo = false, have_hi = false;
            uint32_t delta = stride, th = guess;
            while (c_lo - c_hi > 1 && hi - lo > 1) {
                th = min(max(th, lo + 1), hi - 1);
                const int c = at_least(th, mass);
                if (by_mass ? fm + mass >= target : c >= keep) {
                    lo = th;
                    c_lo = c;
                    have_lo = true;
                    if (!by_mass && c == keep) break;
                } else {
                    hi = th;
                    c_hi = c;
                    have_hi = true;
                }
                if (have_lo && have_hi) {
                    th = lo + (hi - lo) / 2;
                } else {
                    th = have_lo ? lo + min(delta, hi - lo) : hi - min(delta, hi - lo);
                    delta = min(delta, 1u << 28) * 8;
                }
            }
            guess = lo;
            stride = 1u << 18;    // the next row's boundary is within a few percent
            if (hi - lo > 1 || (!by_mass && c_lo == keep)) {
                p = lo - 1;   // exactly the keys from lo up
            } else {
                p = lo;
                if (by_mass) {
                    // the fewest of the equal keys at p that reach the target
                    const int c1 = at_least(p + 1, mass);
                    const double above = fm + mass;
                    const int ties = at_least(p, mass) - c1;
                    const double mp = fmax(static_cast<double>(order_bits_to_float(p)), 0.0);
                    r = 1;
                    while (r < ties && above + static_cast<double>(r) * mp < target) ++r;
                } else {
                    r = keep - c_hi;
                }
            }
        }

        // compaction in ascending j: element by element, block jl + 64 e
        // (the forced test is evaluated again rather than kept as EW lane masks)
        asm volatile("" : "+s"(f0), "+s"(f1), "+s"(f2));
        const size_t orow = (size_t)bh * ldn + i;     // row of the [BH, ldn, ldn] lists
        int32_t* out = kv_idx + orow * ldn;
        int pos = 0, ties = 0;
        auto is_kept = [&](int e) {    // elements in order
            bool kept = vb[e] > p || is_forced(jl + 64 * e);
            if (r > 0) {
                const bool eq = vb[e] == p;
                const uint64_t me = __ballot(eq);
                kept = kept || (eq && ties + mask_rank(me) < r);
                ties += __popcll(me);
            }
            return kept;
        };
        auto put = [&](bool kept, int e) {
            const uint64_t mk = __ballot(kept);
            if (kept) out[pos + mask_rank(mk)] = jl + 64 * e;
            pos += __popcll(mk);
        };
        int total, tid = lane, step = 64;
        if constexpr (SHARED) {
            // the waves hold consecutive blocks: the keys at the boundary, then
            // the kept blocks, of the waves before this one
            if (r > 0) {
                int mine = 0;
#pragma unroll
                for (int e = 0; e < EW; ++e) mine += __popcll(__ballot(vb[e] == p));
                ties = before(mine, total);
            }
            uint32_t km = 0;    // bit e: this lane's block of element e is kept
            int mine = 0;
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                const bool kept = is_kept(e);
                km |= kept ? 1u << e : 0u;
                mine += __popcll(__ballot(kept));
            }
            pos = before(mine, total);
#pragma unroll
            for (int e = 0; e < EW; ++e) put((km >> e) & 1u, e);
            tid = threadIdx.x;
            step = kThreads;
        } else {
#pragma unroll
            for (int e = 0; e < EW; ++e) put(is_kept(e), e);
            total = pos;
        }
        for (int j = n + tid; j < ldn; j += step) out[total + (j - n)] = j;
        if (tid == 0) kv_cnt[orow] = total + (ldn - n);
    }
}

// ---------------------------------------------------------------------------
// a4 + a5, pattern form (Section 5.3): per head, the K largest of the 3n - 1
// predicted pattern intensities (diagonals delta = -(n-1)..n-1 at index
// delta + n - 1, then columns j at 2n - 1 + j), keys at float32 precision,
// ties by pattern index.  One work-group of 1024 threads per head, the order
// bits of its keys in registers (pattern t + 1024 e in element e): it
// extrapolates, finds the K-th largest key by four 8-bit radix passes (each
// a histogram in LDS and a suffix scan of the 256 bins by one wave) and, if
// some but not all of the keys equal to it are chosen, ranks those by index.
// Then per row, block (i, j) is kept iff its diagonal or its column is
// chosen or it is forced; the kept blocks are compacted in ascending j.
// Both are bound by latency and list writes: 24 heads of 929 blocks, K = n/2,
// 9 + 23 us (58 + 74 us with 64-bit keys read again in each of eight passes,
// bins scanned by one thread, and 16 consecutive blocks per thread in the
// rows, whose reads and stores did not coalesce).
// ---------------------------------------------------------------------------
constexpr int kRankThreads = 1024;

__global__ __launch_bounds__(kRankThreads) void pattern_rank_kernel(
    const double* __restrict__ X1, const double* __restrict__ X2, double w, double* __restrict__ pred,
    uint8_t* __restrict__ chosen, int n, int F, int K) {
    constexpr int EP = (3 * kMaxBlocks + kRankThreads - 1) / kRankThreads;
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_digit, s_need, s_ties;
    __shared__ int wcnt[kRankThreads / 64];
    const int P = 3 * n - 1;
    const int bh = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int used = (P + kRankThreads - 1) / kRankThreads;   // elements in use
    uint32_t key[EP];
#pragma unroll
    for (int e = 0; e < EP; ++e) {
        const int q = t + kRankThreads * e;
        key[e] = 0;
        if (q < P) {
            const double v = extrapolated(X1, X2, w, (size_t)bh * (P + F) + q);
            pred[(size_t)bh * P + q] = v;
            key[e] = order_bits(static_cast<float>(v));
        }
    }
    uint32_t prefix = 0, need = (uint32_t)K, ties = 0;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (t < 256) hist[t] = 0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EP; ++e) {
            if (e < used && t + kRankThreads * e < P && (pass == 0 || (key[e] >> (shift + 8)) == prefix))
                atomicAdd(&hist[(key[e] >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (wv == 0) {
            // lane l holds bins 255 - 4l .. 252 - 4l: the largest digits first
            uint32_t b[4], sum = 0;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                b[x] = hist[255 - (4 * lane + x)];
                sum += b[x];
            }
            uint32_t before = wave_inclusive_scan(sum, lane) - sum;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                if (before < need && before + b[x] >= need) {
                    s_digit = 255u - (uint32_t)(4 * lane + x);
                    s_need = need - before;
                    s_ties = b[x];
                }
                before += b[x];
            }
        }
        __syncthreads();
        prefix = (prefix << 8) | s_digit;
        need = s_need;
        ties = s_ties;
    }
    // prefix: the K-th largest key; `need` of the `ties` keys equal to it are chosen
    int before = 0;    // equal keys of smaller index
#pragma unroll
    for (int e = 0; e < EP; ++e) {
        const int q = t + kRankThreads * e;
        const bool eq = q < P && key[e] == prefix;
        bool ch = q < P && (key[e] > prefix || eq);
        if (e < used && need < ties) {
            const uint64_t me = __ballot(eq);
            if (lane == 0) wcnt[wv] = __popcll(me);
            __syncthreads();
            int mine = before, all = 0;
            for (int ww = 0; ww < kRankThreads / 64; ++ww) {
                mine += ww < wv ? wcnt[ww] : 0;
                all += wcnt[ww];
            }
            __syncthreads();
            if (eq) ch = mine + mask_rank(me) < (int)need;
            before += all;
        }
        if (q < P) chosen[(size_t)bh * P + q] = ch ? 1 : 0;
    }
}

__global__ __launch_bounds__(kThreads) void pattern_rows_kernel(
    const uint8_t* __restrict__ chosen, const int32_t* __restrict__ gate,
    const int* __restrict__ row_lo, const int* __restrict__ row_hi, int32_t* __restrict__ kv_idx,
    int32_t* __restrict__ kv_cnt, int n, int ldn, int tb0, int rpw, int chunks) {
    __shared__ uint8_t cs[kMaxBlocks + kWavesPerGroup * kMaxRowsPerWave];   // the rows' diagonals
    __shared__ uint8_t ds[kMaxBlocks];                                      // columns
    const int bh = blockIdx.y;
    if ((int)blockIdx.x >= chunks) {
        keep_all(kv_idx, kv_cnt, (size_t)bh * ldn + tb0 + (blockIdx.x - chunks), ldn);
        return;
    }
    const uint8_t* ch = chosen + (size_t)bh * (3 * n - 1);
    const int i0 = blockIdx.x * kWavesPerGroup * rpw;
    const int i1 = min(n, i0 + kWavesPerGroup * rpw);
    for (int a = threadIdx.x; a < n + (i1 - i0) - 1; a += kThreads) cs[a] = ch[n - i1 + a];
    for (int a = threadIdx.x; a < n; a += kThreads) ds[a] = ch[2 * n - 1 + a];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool g = gate[bh] != 0;
    for (int rr = 0; rr < rpw; ++rr) {
        const int i = i0 + wv * rpw + rr;
        if (i >= min(i1, tb0)) break;
        const int flo = row_lo[i], fhi = row_hi[i];
        const size_t orow = (size_t)bh * ldn + i;     // row of the [BH, ldn, ldn] lists
        int32_t* out = kv_idx + orow * ldn;
        int pos = 0;
        for (int j0 = 0; j0 < n; j0 += 64) {
            const int j = j0 + lane;
            const bool kept = j < n && (cs[j + (i1 - 1 - i)] || ds[j] || (g && j >= flo && j <= fhi) || j == tb0);
            const uint64_t mk = __ballot(kept);
            if (kept) out[pos + mask_rank(mk)] = j;
            pos += __popcll(mk);
        }
        // text blocks after the video blocks: kept in every row
        for (int j = n + lane; j < ldn; j += 64) out[pos + (j - n)] = j;
        if (lane == 0) kv_cnt[orow] = pos + (ldn - n);
    }
}


}  // namespace

hipError_t launch_pool(const uint16_t* q, const uint16_t* k, double* qbar, double* kbar,
                       int BH, int L, int L_stride, int d, int bs, int n, hipStream_t s) {
    const dim3 grid(n, BH, 2);
    if (d == 128 && bs == 128)
        hipLaunchKernelGGL((pool_kernel<128, 128>), grid, dim3(kThreads), 0, s, q, k, qbar, kbar, L, L_stride, n);
    else if (d == 128)
        hipLaunchKernelGGL((pool_kernel<128, 64>), grid, dim3(kThreads), 0, s, q, k, qbar, kbar, L, L_stride, n);
    else if (bs == 128)
        hipLaunchKernelGGL((pool_kernel<64, 128>), grid, dim3(kThreads), 0, s, q, k, qbar, kbar, L, L_stride, n);
    else
        hipLaunchKernelGGL((pool_kernel<64, 64>), grid, dim3(kThreads), 0, s, q, k, qbar, kbar, L, L_stride, n);
    return hipGetLastError();
}

hipError_t launch_logits(const double* qbar, const double* kbar, double* G, int BH, int d, int n, double scale,
                         hipStream_t s) {
    auto go = [&](auto kern, int T) {
        hipLaunchKernelGGL(kern, dim3(cdiv(n, T), cdiv(n, T), (unsigned)BH), dim3(kThreads), 0, s, qbar, kbar, G, n,
                           scale);
        return hipGetLastError();
    };
    // 64 x 64 tiles while they fill the chip twice, else 32 x 32
    const bool fills = (long)BH * cdiv(n, 64) * cdiv(n, 64) >= 512;
    if (d == 128) return fills ? go(logits_kernel<128, 64>, 64) : go(logits_kernel<128, 32>, 32);
    return fills ? go(logits_kernel<64, 64>, 64) : go(logits_kernel<64, 32>, 32);
}

// Rows per work-group of map_sums_kernel: few enough that four work-groups per
// compute unit share a small map's rows (a group's rows are a serial chain),
// 16 otherwise (each chunk adds 2n partial sums to write and read).  4 heads
// of 300 blocks, whole prediction: 83, 67 and 59 us with 32, 16 and 8 rows;
// 24 heads of 929: 574, 565 and 573.
static int sum_rows(int BH, int n) {
    int R = kMaxSumRows;
    while (R > 4 && (long)BH * cdiv(n, R) < 1024) R /= 2;
    return R;
}

// The fit's launch holds a head's whole map in LDS: with up to NC blocks and
// frames, NC = 64 or 128 (0: neither).
static int small_fit(int n, int F) { return std::max(n, F) <= 64 ? 64 : (std::max(n, F) <= 128 ? 128 : 0); }

size_t fit_part_doubles(int BH, int n, int F) {
    if (small_fit(n, F)) return 0;
    const int R = sum_rows(BH, n);
    return (size_t)BH * cdiv(n, R) * (2 * (size_t)n + R - 1);
}

hipError_t launch_fit(double* G, bool logits, const int* reg, const double* Sinv, double* part, double* r, double* bU,
                      double* u, double* X, int BH, int L, int bs, int n, int F, hipStream_t s) {
    // the whole fit in one launch while a head's map fits the LDS
    auto small = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)BH), dim3(kFitThreads), 0, s, G, reg, Sinv, X, L, bs, n, F);
        return hipGetLastError();
    };
    if (small_fit(n, F) == 64) return logits ? small(fit_small_kernel<64, true>) : small(fit_small_kernel<64, false>);
    if (small_fit(n, F) == 128)
        return logits ? small(fit_small_kernel<128, true>) : small(fit_small_kernel<128, false>);

    const int q = n - 1 + F, R = sum_rows(BH, n), nch = (int)cdiv(n, R);
    hipError_t e = hipErrorInvalidValue;
    const int ept = (n + kThreads - 1) / kThreads;
    static_for<1, kMaxBlocks / kThreads + 1>([&](auto w) {
        constexpr int EPT = decltype(w)::value;
        if (ept != EPT) return;
        auto kern = logits ? map_sums_kernel<EPT, true> : map_sums_kernel<EPT, false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)nch, (unsigned)BH), dim3(kThreads), 0, s, G, part, L, bs, n, R);
        e = hipGetLastError();
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rhs_kernel, dim3(cdiv(3 * n - 1, kThreads) + (unsigned)F, (unsigned)BH), dim3(kThreads), 0, s,
                       part, G, reg, r, n, F, nch, R);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(solve_pre_kernel, dim3(cdiv(q, kThreads), BH), dim3(kThreads),
                       (size_t)(2 * n - 1) * sizeof(double), s, r, reg, bU, n, F);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(solve_gemv_kernel, dim3(cdiv(q, 64), kSolveSplit), dim3(kThreads), 0, s, Sinv, bU,
                       u, q, BH);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(solve_post_kernel, dim3(BH), dim3(kPostThreads),
                       (size_t)q * sizeof(double) + (size_t)F * sizeof(int), s, r, u, reg, X, n, F, BH);
    return hipGetLastError();
}

hipError_t launch_gate(const double* Xa, const double* Xb, int32_t* gate, int BH, int n,
                       int F, double tau_e, hipStream_t s) {
    hipLaunchKernelGGL(gate_kernel, dim3(cdiv(BH, 64)), dim3(64), 0, s, Xa, Xb, gate, BH, n, F,
                       tau_e);
    return hipGetLastError();
}

hipError_t launch_select(const double* X1, const double* X2, double w, double* pred, const int32_t* gate,
                         const int* row_lo, const int* row_hi, int mode, int k, double tau, int32_t* kv_idx,
                         int32_t* kv_cnt, int BH, int n, int F, int ldn, int tb0, hipStream_t s) {
    RowGrid rg = row_grid(BH, n, ldn, tb0);
    auto go = [&](auto ew, auto shared) {
        constexpr int EW = decltype(ew)::value;
        constexpr bool SHARED = decltype(shared)::value;
        auto kern = mode == 0 ? select_rows_kernel<EW, false, SHARED> : select_rows_kernel<EW, true, SHARED>;
        hipLaunchKernelGGL(kern, dim3(rg.groups, (unsigned)BH), dim3(kThreads), 0, s, X1, X2, w, pred, gate, row_lo,
                           row_hi, k, tau, kv_idx, kv_cnt, n, F, ldn, tb0, rg.rpw, rg.chunks);
        return hipGetLastError();
    };
    hipError_t e = hipErrorInvalidValue;
    if (n > kWideBlocks) {
        // rows per work-group: as few as give the chip four groups per unit, so
        // that the first row's search and the loads are shared (one head of
        // 4096 blocks, MASS: 106, 105 and 115 us with two, four and eight rows;
        // 8 of 2600: 287, 259, 264)
        rg.rpw = (int)std::max<long>(1, std::min<long>(kMaxSharedRows, (long)BH * n / 1024));
        rg.chunks = (n + rg.rpw - 1) / rg.rpw;
        rg.groups = (unsigned)(rg.chunks + std::max(0, ldn - tb0));
        const int ew = (n + 255) / 256;
        static_for<5, kMaxBlocks / 512 + 1>([&](auto w) {
            constexpr int EW = 2 * decltype(w)::value;
            if (ew <= EW && ew > EW - 2) e = go(std::integral_constant<int, EW>{}, std::true_type{});
        });
        return e;
    }
    // the fewest keys per lane that hold a row (a search step costs one
    // compare per key slot): every width up to 1024 blocks, then every fourth
    const int ew = (n + 63) / 64;
    static_for<1, 17>([&](auto w) {
        if (ew == decltype(w)::value) e = go(w, std::false_type{});
    });
    static_for<5, kWideBlocks / 256 + 1>([&](auto w) {
        constexpr int EW = 4 * decltype(w)::value;
        if (ew > 16 && ew <= EW && ew > EW - 4) e = go(std::integral_constant<int, EW>{}, std::false_type{});
    });
    return e;
}

hipError_t launch_select_patterns(const double* X1, const double* X2, double w, double* pred, const int32_t* gate,
                                  const int* row_lo, const int* row_hi, int K, uint8_t* chosen, int32_t* kv_idx,
                                  int32_t* kv_cnt, int BH, int n, int F, int ldn, int tb0, hipStream_t s) {
    hipLaunchKernelGGL(pattern_rank_kernel, dim3((unsigned)BH), dim3(kRankThreads), 0, s, X1, X2, w, pred, chosen, n,
                       F, K);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const RowGrid rg = row_grid(BH, n, ldn, tb0);
    hipLaunchKernelGGL(pattern_rows_kernel, dim3(rg.groups, (unsigned)BH), dim3(kThreads), 0, s, chosen, gate, row_lo,
                       row_hi, kv_idx, kv_cnt, n, ldn, tb0, rg.rpw, rg.chunks);
    return hipGetLastError();
}

}  // namespace moddit
