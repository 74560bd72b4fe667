// Component-by-component construction of a rank-1 generating vector for the
// weighted Korobov space of smoothness 2 (the P2 criterion of the Korobov
// search, with product weights).  For component s every admissible candidate
// c needs
//   S(c) = sum_{j<n} p_j (1 + w_s B2({j c / n})),   w_s = 2 pi^2 gamma_s,
// with p_j the product over the components already chosen.  B2(1 - x) =
// B2(x), so the point n - j contributes what j does (p_j inherits the
// symmetry from the chosen components), and only j <= n/2 is summed:
// S(c) = 2 sum_{j <= n/2} - term(0) - [n even] term(n/2).  One thread owns
// one candidate and walks its index j c mod n exactly (u32 add and
// conditional subtract); the p_j are staged through LDS in tiles that every
// thread of the block reads in the same order (broadcast reads), and the
// point range is split over grid.y so that small candidate sets still fill
// the chip.  Partial sums are double-double; a second kernel folds them in
// a fixed order, restores the full sum and forms e^2(c) = (S(c) - n) / n.
// The argmin runs on the host, then p_j (j <= n/2) is multiplied by the
// chosen factor.
//
// That direct search costs n^2/4 evaluations per component.  For prime n and
// the full candidate set a convolution screens the candidates first.  With r
// a primitive root and j_t = +-r^t mod n (the class of j_t and n - j_t),
// t < N = (n - 1)/2, the candidate c = j_a has
//   V(c) = sum_{0 < j <= n/2} p_j B2({j c / n}) = sum_t p_{j_t} B2(j_{t+a} / n),
// a cyclic correlation of length N: one FP64 FFT of length L >= 2N - 1 per
// direction gives every V with an error bounded by a multiple of
// log2(L) 2^-53 |p|_2 |B2|_2.  The candidates whose V lies within twice that
// bound plus the tie width of the smallest (one or two of half a million,
// typically) are then summed directly, in the same groups of eight as
// k_cbc_eval, and the choice is made among those exact values by the rule of
// the direct search, so the vector and its errors are the direct search's.
// The whole chain stays on the device; the host reads the result once.
#include <algorithm>
#include <cmath>

#include "qmc_registry.hpp"
#include "qmc_runtime.hpp"

namespace qmc {

namespace {

constexpr uint32_t kCbcTile = 2048;  // doubles of p_j per LDS tile (16 KB)

struct CbcArgs {
    uint32_t n;
    uint32_t jend;    // points j < jend are summed (n/2 + 1)
    uint32_t ncand;
    uint32_t jchunk;  // points per grid.y slice
    double inv_n;
    double w;         // 2 pi^2 gamma_s
    const double *prod;
    const uint32_t *cand;
    double2 *partial;  // [gridDim.y][ncand]
};

__global__ __launch_bounds__(kBlock) void k_cbc_eval(const CbcArgs a) {
    __shared__ double tile[kCbcTile];
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    const bool live = t < a.ncand;
    const uint32_t c = live ? a.cand[t] : 1u;
    const uint32_t j0 = blockIdx.y * a.jchunk;
    const uint32_t j1 = min(a.jend, j0 + a.jchunk);
    dd acc{0.0, 0.0};
    for (uint32_t base = j0; base < j1; base += kCbcTile) {
        const uint32_t cnt = min(kCbcTile, j1 - base);
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < cnt; i += kBlock) tile[i] = a.prod[base + i];
        __syncthreads();
        uint32_t idx = (uint32_t)(((uint64_t)base * c) % a.n);
        // 1 + w B2(x) = w x (x - 1) + (1 + w / 6): two FMAs per point
        const double w6 = 1.0 + a.w / 6.0;
        auto pair = [&](uint32_t i, double &s) {
            const double x = (double)idx * a.inv_n;
            s = fma_(tile[i], fma_(x, fma_(a.w, x, -a.w), w6), s);
            idx += c;
            idx = idx >= a.n ? idx - a.n : idx;
        };
        // groups of 8 points into one plain sum, then the double-double fold
        // (written as a loop over whole groups: a fold guarded inside the
        // point loop was if-converted and ran at every unrolled step)
        uint32_t i = 0;
        for (; i + 8 <= cnt; i += 8) {
            double s = 0.0;
#pragma unroll
            for (uint32_t u = 0; u < 8; ++u) pair(i + u, s);
            dd_accumulate(acc.hi, acc.lo, s);
        }
        double s = 0.0;
        for (; i < cnt; ++i) pair(i, s);
        dd_accumulate(acc.hi, acc.lo, s);
    }
    if (live) a.partial[(size_t)blockIdx.y * a.ncand + t] = make_double2(acc.hi, acc.lo);
}

// e2[t] = (S - n) / n with S = 2 (sum over slices) - term(0) - [n even]
// term(n/2), slices folded in order; the two terms are formed as k_cbc_eval
// forms them (x = idx / n through inv_n)
__global__ __launch_bounds__(kBlock) void k_cbc_reduce(const double2 *partial, uint32_t slices, uint32_t ncand,
                                                       uint32_t n, double inv_n, double w, const double *prod,
                                                       double *e2) {
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= ncand) return;
    dd acc{0.0, 0.0};
    for (uint32_t y = 0; y < slices; ++y) {
        const double2 v = partial[(size_t)y * ncand + t];
        acc = dd_add(acc, dd{v.x, v.y});
    }
    acc = dd{2.0 * acc.hi, 2.0 * acc.lo};
    const double w6 = 1.0 + w / 6.0;
    acc = dd_add(acc, dd{-(prod[0] * w6), 0.0});
    if ((n & 1u) == 0) {  // j = n/2 is its own mirror; c is odd, so idx = n/2
        const double x = (double)(n / 2) * inv_n;
        acc = dd_add(acc, dd{-(prod[n / 2] * fma_(x, fma_(w, x, -w), w6)), 0.0});
    }
    e2[t] = ((acc.hi - (double)n) + acc.lo) / (double)n;
}

// p_j *= 1 + w B2({j z / n}) for j < jend
__global__ __launch_bounds__(kBlock) void k_cbc_update(double *prod, uint32_t n, uint32_t jend, double inv_n,
                                                       uint32_t z, double w) {
    const uint32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= jend) return;
    const uint32_t idx = (uint32_t)(((uint64_t)j * z) % n);
    const double x = (double)idx * inv_n;
    prod[j] = prod[j] * fma_(w, fma_(x, x - 1.0, 1.0 / 6.0), 1.0);
}

__global__ __launch_bounds__(kBlock) void k_fill(double *p, uint32_t count, double v) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < count) p[i] = v;
}

// ------------------------------------------------- screening by convolution
// L = 2^(LOG1 + LOG2) points as an M1 x M2 matrix (M1 = 2^LOG1 rows).
// k_cbc_col transforms columns (stride M2, kCols neighbouring columns per
// workgroup so that a row segment is 32-64 bytes) and applies the twiddle
// factors exp(-2 pi i n2 k1 / L); k_cbc_row transforms the contiguous rows
// and, for p, multiplies by the stored spectrum of B2 and transforms back in
// the same pass (the product needs no particular order, so no transpose is
// ever made); k_cbc_col_inv undoes the columns and keeps the smallest V of
// each workgroup.  Inside a workgroup the transform runs in LDS as radix-4
// Stockham steps (4 columns: 64 KB at L = 2^20, two workgroups per CU).  A
// component is three passes over 16 L bytes, which stay in the last-level
// cache at n = 2^20 - 3 (L = 2^20): 17, 21 and 13 us, bound by the LDS steps
// and their barriers, and four launches of 4-8 us for the selection, the
// finalists' sums, the choice and the update of p.  The whole search at
// d = 10 takes 0.87 ms there (635 ms by direct sums alone), 0.49 ms at
// n = 131071 (13 ms) and 0.36 ms at n = 16381 (1.3 ms).
constexpr int kCbcTw = 4096;          // entries of the step twiddle table exp(-2 pi i t / 4096)
constexpr uint32_t kCbcFinal = 1024;  // finalists summed directly; more fall back to the direct search
constexpr uint32_t kCbcUpd = 256;     // workgroups of k_cbc_advance (partial sums of p)

constexpr double two_pi2 = 2.0 * 3.141592653589793 * 3.141592653589793;

struct CbcState {
    uint32_t count;     // finalists of the component at hand
    uint32_t overflow;  // 1 + the component whose finalists did not fit (0: none)
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(fma_(a.x, b.x, -(a.y * b.y)), fma_(a.x, b.y, a.y * b.x));
}

// exp(-2 pi i e / 2^log), conjugated for the inverse
template <bool Inv>
__device__ __forceinline__ double2 cbc_root(uint32_t e, int log) {
    double sn, cs;
    sincospi(__builtin_amdgcn_ldexp((double)e, 1 - log), &sn, &cs);
    return make_double2(cs, Inv ? sn : -sn);
}

// The transforms of CW interleaved sequences of 2^LOG points in LDS (point i
// of sequence c at s[i CW + c]), natural order in and out, by NT threads.
template <int LOG, int CW, int NT, bool Inv>
__device__ __forceinline__ void cbc_fft(double2 *s, const double2 *__restrict__ tw) {
    constexpr int M = 1 << LOG;
    constexpr int N4 = M / 4 * CW, B4 = (N4 + NT - 1) / NT;
    const int tid = (int)threadIdx.x;
    int p = 1;
#pragma unroll 1
    for (; p * 4 <= M; p *= 4) {
        double2 u[B4][4];
#pragma unroll
        for (int b = 0; b < B4; ++b) {
            const int id = tid + b * NT;
            if (id < N4) {
#pragma unroll
                for (int q = 0; q < 4; ++q) u[b][q] = s[id + q * N4];
            }
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B4; ++b) {
            const int id = tid + b * NT;
            if (id < N4) {
                const int c = id % CW, i = id / CW, k = i & (p - 1), j = ((i - k) << 2) + k;
                const int ts = k * (kCbcTw / 4 / p);
#pragma unroll
                for (int q = 1; q < 4; ++q) {
                    double2 w = tw[q * ts];
                    if (Inv) w.y = -w.y;
                    u[b][q] = cmul(u[b][q], w);
                }
                const double2 v0 = make_double2(u[b][0].x + u[b][2].x, u[b][0].y + u[b][2].y);
                const double2 v1 = make_double2(u[b][0].x - u[b][2].x, u[b][0].y - u[b][2].y);
                const double2 v2 = make_double2(u[b][1].x + u[b][3].x, u[b][1].y + u[b][3].y);
                const double2 d = make_double2(u[b][1].x - u[b][3].x, u[b][1].y - u[b][3].y);
                const double2 v3 = Inv ? make_double2(-d.y, d.x) : make_double2(d.y, -d.x);  // -+ i d
                s[(j)*CW + c] = make_double2(v0.x + v2.x, v0.y + v2.y);
                s[(j + p) * CW + c] = make_double2(v1.x + v3.x, v1.y + v3.y);
                s[(j + 2 * p) * CW + c] = make_double2(v0.x - v2.x, v0.y - v2.y);
                s[(j + 3 * p) * CW + c] = make_double2(v1.x - v3.x, v1.y - v3.y);
            }
        }
        __syncthreads();
    }
    if constexpr (LOG & 1) {
        constexpr int N2 = M / 2 * CW, B2 = (N2 + NT - 1) / NT;
        double2 u[B2][2];
#pragma unroll
        for (int b = 0; b < B2; ++b) {
            const int id = tid + b * NT;
            if (id < N2) {
                u[b][0] = s[id];
                u[b][1] = s[id + N2];
            }
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < B2; ++b) {
            const int id = tid + b * NT;
            if (id < N2) {  // p = M / 2 here, so k = i and j = i
                const int i = id / CW;
                double2 w = tw[i * (kCbcTw / M)];
                if (Inv) w.y = -w.y;
                const double2 t = cmul(u[b][1], w);
                s[id] = make_double2(u[b][0].x + t.x, u[b][0].y + t.y);
                s[id + N2] = make_double2(u[b][0].x - t.x, u[b][0].y - t.y);
            }
        }
        __syncthreads();
    }
}

struct CbcFftArgs {
    uint32_t n, N;         // lattice size (prime), (n - 1) / 2
    double inv_n;
    const uint32_t *perm;  // j_t, t < N
    const double *prod;    // p_j (null: transform B2)
    const double2 *tw;
    double2 *work;         // (M1, M2)
    const double2 *spec;   // spectrum of B2, in k_cbc_row's layout
    double *value;         // V of candidate j_a at a
    double *vmin;          // smallest V of each workgroup of k_cbc_col_inv
    CbcState *state;
};

constexpr int cbc_cols(int log1) { return log1 <= 10 ? 4 : 2; }  // at most 64 KB of LDS
constexpr int kCbcColThreads = 512, kCbcRowThreads = 256;

template <int LOG1, int LOG2>
__global__ __launch_bounds__(kCbcColThreads) void k_cbc_col(const CbcFftArgs a) {
    constexpr int M1 = 1 << LOG1, M2 = 1 << LOG2, CW = cbc_cols(LOG1);
    __shared__ double2 s[M1 * CW];
    const uint32_t c0 = blockIdx.x * CW, stop = a.state->overflow;  // looked at behind the loads
    if (blockIdx.x == 0 && threadIdx.x == 0) a.state->count = 0;
    for (uint32_t e = threadIdx.x; e < (uint32_t)(M1 * CW); e += kCbcColThreads) {
        const uint32_t t = (e / CW) * M2 + c0 + e % CW;
        double v = 0.0;
        if (a.prod) {
            if (t < a.N) v = a.prod[a.perm[t]];
        } else if (t < 2 * a.N - 1) {  // B2 continued periodically: 2N - 1 values
            const double x = (double)a.perm[t < a.N ? t : t - a.N] * a.inv_n;
            v = fma_(x, x - 1.0, 1.0 / 6.0);
        }
        s[e] = make_double2(v, 0.0);
    }
    if (stop) return;
    __syncthreads();
    cbc_fft<LOG1, CW, kCbcColThreads, false>(s, a.tw);
    for (uint32_t e = threadIdx.x; e < (uint32_t)(M1 * CW); e += kCbcColThreads) {
        const uint32_t k1 = e / CW, n2 = c0 + e % CW;
        a.work[(size_t)k1 * M2 + n2] = cmul(s[e], cbc_root<false>(k1 * n2, LOG1 + LOG2));
    }
}

template <int LOG1, int LOG2>
__global__ __launch_bounds__(kCbcRowThreads) void k_cbc_row(const CbcFftArgs a) {
    constexpr int M2 = 1 << LOG2;
    __shared__ double2 s[M2];
    const uint32_t k1 = blockIdx.x, stop = a.state->overflow;
    double2 *row = a.work + (size_t)k1 * M2;
    for (uint32_t e = threadIdx.x; e < (uint32_t)M2; e += kCbcRowThreads) s[e] = row[e];
    if (stop) return;
    __syncthreads();
    cbc_fft<LOG2, 1, kCbcRowThreads, false>(s, a.tw);
    if (!a.prod) {  // the spectrum of B2 itself
        for (uint32_t e = threadIdx.x; e < (uint32_t)M2; e += kCbcRowThreads) row[e] = s[e];
        return;
    }
    for (uint32_t e = threadIdx.x; e < (uint32_t)M2; e += kCbcRowThreads) {
        const double2 f = s[e];
        s[e] = cmul(make_double2(f.x, -f.y), a.spec[(size_t)k1 * M2 + e]);
    }
    __syncthreads();
    cbc_fft<LOG2, 1, kCbcRowThreads, true>(s, a.tw);
    for (uint32_t e = threadIdx.x; e < (uint32_t)M2; e += kCbcRowThreads)
        row[e] = cmul(s[e], cbc_root<true>(k1 * e, LOG1 + LOG2));
}

template <int LOG1, int LOG2>
__global__ __launch_bounds__(kCbcColThreads) void k_cbc_col_inv(const CbcFftArgs a) {
    constexpr int M1 = 1 << LOG1, M2 = 1 << LOG2, CW = cbc_cols(LOG1);
    __shared__ double2 s[M1 * CW];
    const uint32_t c0 = blockIdx.x * CW, stop = a.state->overflow;
    for (uint32_t e = threadIdx.x; e < (uint32_t)(M1 * CW); e += kCbcColThreads)
        s[e] = a.work[(size_t)(e / CW) * M2 + c0 + e % CW];
    if (stop) return;
    __syncthreads();
    cbc_fft<LOG1, CW, kCbcColThreads, true>(s, a.tw);
    double lo = __builtin_inf();
    for (uint32_t e = threadIdx.x; e < (uint32_t)(M1 * CW); e += kCbcColThreads) {
        const uint32_t t = (e / CW) * M2 + c0 + e % CW;
        if (t < a.N) {
            const double v = s[e].x * (1.0 / ((double)M1 * M2));
            a.value[t] = v;
            lo = __builtin_fmin(lo, v);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lo = __builtin_fmin(lo, __shfl_xor(lo, off, kWave));
    __syncthreads();  // s has been read
    if ((threadIdx.x & (kWave - 1)) == 0) s[threadIdx.x / kWave].x = lo;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kCbcColThreads / kWave; ++w) lo = __builtin_fmin(lo, s[w].x);
        a.vmin[blockIdx.x] = lo;
    }
}

// step twiddles and the classes j_t (r^t by repeated squaring)
__global__ __launch_bounds__(kBlock) void k_cbc_tables(double2 *tw, uint32_t *perm, uint32_t n, uint32_t N,
                                                       double inv_n, uint32_t root) {
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    if (t < (uint32_t)kCbcTw) tw[t] = cbc_root<false>(t, 12);
    if (t >= N) return;
    uint32_t v = 1, b = root;
    for (uint32_t e = t; e; e >>= 1) {
        if (e & 1u) v = mulmod(v, b, n, inv_n);
        b = mulmod(b, b, n, inv_n);
    }
    perm[t] = min(v, n - v);
}

// candidates whose V lies within the slack of the smallest
struct CbcSelectArgs {
    uint32_t n, N, nmin;
    double w, tol;           // tol: the transform's error per |p|_2 (the host's bound)
    const double *value, *vmin, *prod;
    const double2 *psum;     // per workgroup of k_cbc_advance: sum p, sum p^2 (j >= 1)
    const uint32_t *perm;
    uint32_t *list;
    CbcState *state;
};

__global__ __launch_bounds__(kBlock) void k_cbc_select(const CbcSelectArgs a) {
    __shared__ double red[3][kBlock / kWave];
    double lo = __builtin_inf(), s1 = 0.0, s2 = 0.0;
    for (uint32_t i = threadIdx.x; i < a.nmin; i += kBlock) lo = __builtin_fmin(lo, a.vmin[i]);
    for (uint32_t i = threadIdx.x; i < kCbcUpd; i += kBlock) {
        s1 += a.psum[i].x;
        s2 += a.psum[i].y;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = __builtin_fmin(lo, __shfl_xor(lo, off, kWave));
        s1 += __shfl_xor(s1, off, kWave);
        s2 += __shfl_xor(s2, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][threadIdx.x / kWave] = lo;
        red[1][threadIdx.x / kWave] = s1;
        red[2][threadIdx.x / kWave] = s2;
    }
    __syncthreads();
    s1 = s2 = 0.0;
    for (int w = 0; w < kBlock / kWave; ++w) {
        lo = __builtin_fmin(lo, red[0][w]);
        s1 += red[1][w];
        s2 += red[2][w];
    }
    // e^2 of the smallest, the tie width around it, and the rounding of the
    // direct sums (16 ulp of sum |p_j| (1 + w/6) <= sqrt(N sum p^2) (1 + w/6))
    const double nn = (double)a.n, w6 = 1.0 + a.w / 6.0;
    const double e2 = (2.0 * (s1 + a.w * lo) + a.prod[0] * w6 - nn) / nn;
    const double tie = 1.01e-13 * (1.0 + __builtin_fabs(e2));
    const double direct = 16.0 * 0x1p-52 * w6 * __builtin_sqrt((double)a.N * s2) / nn;
    const double thr = lo + 2.0 * a.tol * __builtin_sqrt(s2) + (tie + 2.0 * direct) * nn / (2.0 * a.w);
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    if (t < a.N && a.value[t] <= thr) {
        const uint32_t at = atomicAdd(&a.state->count, 1u);
        if (at < kCbcFinal) a.list[at] = a.perm[t];
    }
}

// Direct sums of the finalists.  A workgroup owns one tile of kCbcTile points
// of one slice (the tiles of k_cbc_eval with `slices` slices of jchunk
// points), each thread one of its groups of 8, and walks the finalists
// (blockIdx.y, blockIdx.y + gridDim.y, ...).
__global__ __launch_bounds__(kBlock) void k_cbc_exact(const CbcArgs a, uint32_t tiles, const CbcState *state) {
    static_assert(kCbcTile == 8 * kBlock, "one group of 8 per thread");
    __shared__ dd red[kBlock / kWave];
    const uint32_t y = blockIdx.x / tiles, q = blockIdx.x - y * tiles;
    const uint32_t j0 = y * a.jchunk, j1 = min(a.jend, j0 + a.jchunk);
    const uint32_t first = j0 + q * kCbcTile + 8 * threadIdx.x;
    const uint32_t cnt = first < j1 ? min(8u, j1 - first) : 0u;
    double p[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) p[u] = u < cnt ? a.prod[first + u] : 0.0;
    const double w6 = 1.0 + a.w / 6.0;
    // finalists that do not fit are left to the direct search
    const uint32_t nf = state->overflow || state->count > kCbcFinal ? 0u : state->count;
    for (uint32_t f = blockIdx.y; f < nf; f += gridDim.y) {
        const uint32_t c = a.cand[f];
        uint32_t idx = cnt ? (uint32_t)(((uint64_t)first * c) % a.n) : 0u;
        double s = 0.0;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const double x = (double)idx * a.inv_n;
            const double t = fma_(p[u], fma_(x, fma_(a.w, x, -a.w), w6), s);
            s = u < cnt ? t : s;
            idx += c;
            idx = idx >= a.n ? idx - a.n : idx;
        }
        const dd r = wave_reduce(dd{s, 0.0});
        __syncthreads();
        if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = r;
        __syncthreads();
        if (threadIdx.x == 0) {
            dd t = red[0];
            for (int w = 1; w < kBlock / kWave; ++w) t = dd_add(t, red[w]);
            a.partial[(size_t)f * gridDim.x + blockIdx.x] = make_double2(t.hi, t.lo);
        }
    }
}

// e^2 of the finalists as k_cbc_reduce forms it, then the choice: the
// smallest c within the tie width of the smallest e^2
__global__ __launch_bounds__(1024) void k_cbc_choose(const double2 *partial, uint32_t nparts, uint32_t n, double inv_n,
                                                     double w, const double *prod, const uint32_t *list,
                                                     CbcState *state, uint32_t comp, uint32_t *z, double *e2) {
    __shared__ double h[kCbcFinal];
    const uint32_t nf = state->count, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (state->overflow) return;
    if (nf == 0 || nf > kCbcFinal) {  // none: the values are not finite
        if (threadIdx.x == 0) state->overflow = comp + 1;
        return;
    }
    const double w6 = 1.0 + w / 6.0;
    for (uint32_t f = wave; f < nf; f += 1024 / kWave) {
        dd acc{0.0, 0.0};
        for (uint32_t i = lane; i < nparts; i += kWave) {
            const double2 v = partial[(size_t)f * nparts + i];
            acc = dd_add(acc, dd{v.x, v.y});
        }
        acc = wave_reduce(acc);
        if (lane == 0) {
            acc = dd{2.0 * acc.hi, 2.0 * acc.lo};
            acc = dd_add(acc, dd{-(prod[0] * w6), 0.0});
            h[f] = ((acc.hi - (double)n) + acc.lo) / (double)n;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double vmin = h[0];
        for (uint32_t f = 1; f < nf; ++f) vmin = __builtin_fmin(vmin, h[f]);
        const double lim = vmin + 1e-13 * (1.0 + __builtin_fabs(vmin));
        uint32_t best = 0xffffffffu;
        double eb = vmin;
        for (uint32_t f = 0; f < nf; ++f)
            if (h[f] <= lim && lim < __builtin_inf() && list[f] < best) {
                best = list[f];
                eb = h[f];
            }
        if (best == 0xffffffffu) {  // not finite: left to the direct search
            state->overflow = comp + 1;
        } else {
            z[comp] = best;
            e2[comp] = eb;
        }
    }
}

// k_cbc_update with the chosen component, and the sums of p and p^2 (j >= 1)
// (z: where k_cbc_choose left it, or null for the component zv)
__global__ __launch_bounds__(kBlock) void k_cbc_advance(double *prod, uint32_t n, uint32_t jend, double inv_n,
                                                        const uint32_t *z, uint32_t zv, double w,
                                                        const CbcState *state, double2 *psum) {
    __shared__ double red[2][kBlock / kWave];
    if (state->overflow) return;
    const uint32_t c = z ? *z : zv;
    double s1 = 0.0, s2 = 0.0;
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < jend; j += kCbcUpd * kBlock) {
        const uint32_t idx = (uint32_t)(((uint64_t)j * c) % n);
        const double x = (double)idx * inv_n;
        const double p = prod[j] * fma_(w, fma_(x, x - 1.0, 1.0 / 6.0), 1.0);
        prod[j] = p;
        if (j) {
            s1 += p;
            s2 = fma_(p, p, s2);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s1 += __shfl_xor(s1, off, kWave);
        s2 += __shfl_xor(s2, off, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        red[0][threadIdx.x / kWave] = s1;
        red[1][threadIdx.x / kWave] = s2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < kBlock / kWave; ++v) {
            s1 += red[0][v];
            s2 += red[1][v];
        }
        psum[blockIdx.x] = make_double2(s1, s2);
    }
}

template <int LOG1, int LOG2>
void cbc_launch_fft(const CbcFftArgs &a, bool forward_only) {
    constexpr uint32_t cols = (1u << LOG2) / cbc_cols(LOG1);
    hipLaunchKernelGGL((k_cbc_col<LOG1, LOG2>), dim3(cols), dim3(kCbcColThreads), 0, nullptr, a);
    hipLaunchKernelGGL((k_cbc_row<LOG1, LOG2>), dim3(1u << LOG1), dim3(kCbcRowThreads), 0, nullptr, a);
    if (!forward_only)
        hipLaunchKernelGGL((k_cbc_col_inv<LOG1, LOG2>), dim3(cols), dim3(kCbcColThreads), 0, nullptr, a);
}

// log2 of the transform length: the smallest power of two >= 2N - 1 = n - 2.
// The bound on the work (n/2 candidates x n <= 2^44) keeps n below 2^23.
constexpr int kCbcLogMin = 14, kCbcLogMax = 23;
int cbc_log(uint64_t n) {
    int l = kCbcLogMin;
    while ((1ull << l) < n - 2) ++l;
    return l;
}

void cbc_fft_pass(int log, const CbcFftArgs &a, bool forward_only) {
    switch (log) {
    case 14: return cbc_launch_fft<7, 7>(a, forward_only);
    case 15: return cbc_launch_fft<7, 8>(a, forward_only);
    case 16: return cbc_launch_fft<8, 8>(a, forward_only);
    case 17: return cbc_launch_fft<8, 9>(a, forward_only);
    case 18: return cbc_launch_fft<9, 9>(a, forward_only);
    case 19: return cbc_launch_fft<9, 10>(a, forward_only);
    case 20: return cbc_launch_fft<10, 10>(a, forward_only);
    case 21: return cbc_launch_fft<10, 11>(a, forward_only);
    case 22: return cbc_launch_fft<11, 11>(a, forward_only);
    default: return cbc_launch_fft<11, 12>(a, forward_only);
    }
}

// workgroups of k_cbc_col_inv (entries of vmin)
uint32_t cbc_col_groups(int log) {
    const int log1 = log / 2;
    return (1u << (log - log1)) / cbc_cols(log1);
}

// the distinct prime factors of v
std::vector<uint64_t> prime_factors(uint64_t v) {
    std::vector<uint64_t> f;
    for (uint64_t p = 2; p * p <= v; ++p)
        if (v % p == 0) {
            f.push_back(p);
            while (v % p == 0) v /= p;
        }
    if (v > 1) f.push_back(v);
    return f;
}

uint64_t pow_mod(uint64_t b, uint64_t e, uint64_t n) {
    uint64_t r = 1;
    for (; e; e >>= 1, b = b * b % n)
        if (e & 1) r = r * b % n;
    return r;
}

// smallest primitive root of a prime n < 2^32
uint64_t primitive_root(uint64_t n) {
    const std::vector<uint64_t> f = prime_factors(n - 1);
    for (uint64_t g = 2;; ++g) {
        bool ok = true;
        for (uint64_t p : f) ok = ok && pow_mod(g, (n - 1) / p, n) != 1;
        if (ok) return g;
    }
}

// Smallest prime n that is screened: with d = 10 the screened search takes
// 344, 341, 343, 354 us at n = 509, 1021, 2039, 4099 (launches; the transform
// is 2^14 points there), the direct one 335, 404, 538, 909 us.
constexpr uint64_t kScreenMin = 1000;

// How far apart the errors of a component's candidates lie, to within a
// factor of a few: P, the product of its weight and the largest one before it
// over n^2.  The share of the candidates within the tie width of the best
// follows it, about 1e-14 / P: 0.1 % at 1e-11, 1 % at 1e-12, 20 to 25 % at 2e-13,
// 73 % at 2e-14, 93 % at 2e-15 (n = 2039, 4099, 16381).  Many ties are too many
// finalists, and then the component is summed directly after all.  So:
// - below kTieSure, where no screening pays, a component is not screened if
//   the direct search is cheap (below kTieDirect points 50 to 300 us a
//   component, the screening 40 to 60 us); nor with equal errors (0), nor
//   after a component with a wider spread that had too many ties;
// - below kTieLook times the candidates it is screened and the host looks at
//   the outcome before it enqueues the next (half of what makes 1024 finalists
//   by the share above: P is low where several weights are near the largest,
//   and a look costs 10 us);
// - above, every component is enqueued ahead; one that has too many finalists
//   all the same wastes the launches behind it, which return at once;
// - where all candidates fit the finalists' list (n < 2048), screened and direct
//   components are not mixed: the direct search of one takes 40 us there, no
//   more than the buffers and tables of the screening.
// Trailing zero weights, or weights of 1e-9, at n = 4099, d = 10: 0.77 ms (13 ms
// when every component was screened first and all behind it enqueued again
// after each that had too many ties; 0.80 ms by direct sums alone); at n = 16381
// 0.98, 13.2 and 1.10 ms.
constexpr double kTieSure = 5e-13, kTieLook = 5e-18;
constexpr uint64_t kTieDirect = 32768;

double cbc_spread(const std::vector<double> &gam, uint32_t c, uint64_t n) {
    const double w = two_pi2 * gam[c], top = two_pi2 * *std::max_element(gam.begin(), gam.begin() + c);
    return w / (double)n * (top / (double)n);
}

// tied: the largest spread that had too many ties so far
bool cbc_unscreened(double spread, double tied, uint64_t n) {
    return spread <= tied || (spread < kTieSure && n < kTieDirect);
}

uint64_t gcd_u64(uint64_t a, uint64_t b) {
    while (b) {
        const uint64_t r = a % b;
        a = b;
        b = r;
    }
    return a;
}

}  // namespace
}  // namespace qmc

using namespace qmc;

extern "C" qmc_status qmc_cbc_search(uint64_t n, uint32_t d, const double *gamma, const uint64_t *cand,
                                     uint32_t ncand, uint64_t *z_out, double *e2_out) {
    if (!z_out || !e2_out) return fail(QMC_EINVAL, "null output");
    if (d == 0) return fail(QMC_EINVAL, "d must be >= 1");
    if (d > kMaxDim) return fail(QMC_EUNSUPPORTED, "d > %u", kMaxDim);
    if (n < 2) return fail(QMC_EINVAL, "n must be >= 2");
    if (n > (1ull << 31)) return fail(QMC_EUNSUPPORTED, "n > 2^31");
    std::vector<double> gam(d, 1.0);
    if (gamma)
        for (uint32_t i = 0; i < d; ++i) {
            if (!(gamma[i] >= 0.0) || !std::isfinite(gamma[i])) return fail(QMC_EINVAL, "gamma_%u not finite or < 0", i);
            gam[i] = gamma[i];
        }
    std::vector<uint32_t> cs;
    bool screen = false;
    if (cand) {
        if (ncand == 0) return fail(QMC_EINVAL, "ncand must be >= 1");
        for (uint32_t t = 0; t < ncand; ++t) {
            if (cand[t] == 0 || cand[t] >= n || gcd_u64(cand[t], n) != 1)
                return fail(QMC_EINVAL, "candidate %u is not a unit mod n", t);
            cs.push_back((uint32_t)cand[t]);
        }
        std::sort(cs.begin(), cs.end());
        cs.erase(std::unique(cs.begin(), cs.end()), cs.end());
    } else {
        // every unit up to n/2: bound the work before enumerating them
        if ((double)(n / 2) * (double)n > 17592186044416.0)
            return fail(QMC_EUNSUPPORTED, "n/2 candidates x n = %.3g > 2^44: pass a candidate subset",
                        (double)(n / 2) * (double)n);
        // screened search (above): prime n from kScreenMin up
        const std::vector<uint64_t> pf = prime_factors(n);
        screen = n >= kScreenMin && pf.size() == 1 && pf[0] == n && cbc_log(n) <= kCbcLogMax;
        const bool prime = screen;
        if (screen && d > 1) {
            uint32_t count = 0;
            for (uint32_t c = 1; c < d; ++c) count += !cbc_unscreened(cbc_spread(gam, c, n), 0.0, n);
            screen = n / 2 > kCbcFinal ? count > 0 : count == d - 1;
        }
        if (!screen) {
            for (uint64_t c = 1; c <= n / 2; ++c)
                if (prime || gcd_u64(c, n) == 1) cs.push_back((uint32_t)c);
            if (cs.empty()) cs.push_back(1u);
        }
    }
    // keep the cost of one component within a few seconds
    if (!screen && (double)cs.size() * (double)n > 17592186044416.0)
        return fail(QMC_EUNSUPPORTED, "candidates x n = %.3g > 2^44: pass a candidate subset", (double)cs.size() * (double)n);
    const uint32_t nc = screen ? (uint32_t)(n / 2) : (uint32_t)cs.size();
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    const uint32_t want = 8u * (uint32_t)device_cu_count(dev);
    const uint32_t jend = (uint32_t)(n / 2 + 1);  // j <= n/2 (mirror symmetry j <-> n - j)
    const uint32_t max_slices = std::max<uint32_t>(1, jend / kCbcTile);
    const uint32_t bx = (nc + kBlock - 1) / kBlock;
    const uint32_t slices = std::min(max_slices, std::max(1u, (want + bx - 1) / bx));
    const uint32_t nb = (jend + kBlock - 1) / kBlock;
    const double inv_n = 1.0 / (double)n;
    DeviceScratch s;
    qmc_status st;

    // the direct search's buffers, made when it first runs
    uint32_t *dcand = nullptr;
    double2 *dpartial = nullptr;
    double *de2 = nullptr;
    std::vector<double> h;
    // component comp by direct sums over every candidate
    auto direct = [&](uint32_t comp, double *prod) -> qmc_status {
        const double w = two_pi2 * gam[comp];
        // z_1 = 1: in one dimension every unit gives the same point set
        const bool first = comp == 0;
        if (!dcand) {
            if (cs.empty())  // a prime n, screened so far: every c <= n/2 is a unit
                for (uint32_t c = 1; c <= nc; ++c) cs.push_back(c);
            h.resize(nc);
            const uint32_t one_h = 1u;
            // candidates, then the single candidate of the first component
            if ((st = s.alloc((size_t)nc * 4 + 4)) || (st = s.alloc(((size_t)slices * nc + want) * sizeof(double2))) ||
                (st = s.alloc((size_t)nc * 8)))
                return st;
            const size_t at = s.ptr.size() - 3;
            dcand = (uint32_t *)s.ptr[at];
            dpartial = (double2 *)s.ptr[at + 1];
            de2 = (double *)s.ptr[at + 2];
            if ((e = hipMemcpy(dcand, cs.data(), (size_t)nc * 4, hipMemcpyHostToDevice)) != hipSuccess ||
                (e = hipMemcpy(dcand + nc, &one_h, 4, hipMemcpyHostToDevice)) != hipSuccess)
                return hip_fail(e, "cbc upload");
        }
        const uint32_t cnt = first ? 1u : nc;
        const uint32_t cbx = first ? 1u : bx;
        const uint32_t csl = first ? std::min(max_slices, want) : slices;
        const uint32_t cch = (jend + csl - 1) / csl;
        CbcArgs a{(uint32_t)n, jend, cnt, cch, inv_n, w, prod, first ? dcand + nc : dcand, dpartial};
        hipLaunchKernelGGL(k_cbc_eval, dim3(cbx, csl), dim3(kBlock), 0, nullptr, a);
        hipLaunchKernelGGL(k_cbc_reduce, dim3((cnt + kBlock - 1) / kBlock), dim3(kBlock), 0, nullptr,
                           (const double2 *)dpartial, csl, cnt, (uint32_t)n, inv_n, w, (const double *)prod, de2);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch CBC kernels");
        if ((e = hipMemcpy(h.data(), de2, (size_t)cnt * 8, hipMemcpyDeviceToHost)) != hipSuccess)
            return hip_fail(e, "cbc download");
        // lattice symmetries make exact ties common (in two dimensions c and
        // c^-1 mod n give the same error) and rounding would choose among
        // them: values within 1e-13 (1 + e^2) of the minimum are ties, and
        // ties go to the smallest c (candidates ascend)
        double vmin = h[0];
        for (uint32_t t = 1; t < cnt; ++t) vmin = std::min(vmin, h[t]);
        if (!std::isfinite(vmin)) return fail(QMC_ENONFINITE, "CBC error not finite");
        const double tau = 1e-13 * (1.0 + std::fabs(vmin));
        uint32_t best = 0;
        while (!(h[best] <= vmin + tau)) ++best;
        z_out[comp] = first ? 1u : cs[best];
        e2_out[comp] = h[best];
        return QMC_OK;
    };

    if (!screen) {
        if ((st = s.alloc((size_t)jend * 8))) return st;
        double *prod = (double *)s.ptr[0];
        hipLaunchKernelGGL(k_fill, dim3(nb), dim3(kBlock), 0, nullptr, prod, jend, 1.0);
        for (uint32_t comp = 0; comp < d; ++comp) {
            if ((st = direct(comp, prod))) return st;
            hipLaunchKernelGGL(k_cbc_update, dim3(nb), dim3(kBlock), 0, nullptr, prod, (uint32_t)n, jend, inv_n,
                               (uint32_t)z_out[comp], two_pi2 * gam[comp]);
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch CBC update");
        }
        if ((e = hipDeviceSynchronize()) != hipSuccess) return hip_fail(e, "cbc synchronize");
        return QMC_OK;
    }

    // one allocation, cut into 256-byte aligned parts
    const int log = cbc_log(n);
    const uint32_t N = (uint32_t)((n - 1) / 2), L = 1u << log;
    // tiles of a slice: the first component and the others cut their slices differently
    const uint32_t sl1 = std::min(max_slices, want), ch1 = (jend + sl1 - 1) / sl1, chs = (jend + slices - 1) / slices;
    const uint32_t t1 = (ch1 + kCbcTile - 1) / kCbcTile, ts = (chs + kCbcTile - 1) / kCbcTile;
    size_t total = 0;
    auto part = [&](size_t bytes) {
        const size_t at = total;
        total += (bytes + 255) / 256 * 256;
        return at;
    };
    const size_t o_prod = part((size_t)jend * 8), o_perm = part((size_t)N * 4), o_tw = part(kCbcTw * 16),
                 o_spec = part((size_t)L * 16), o_work = part((size_t)L * 16), o_value = part((size_t)N * 8),
                 o_vmin = part((size_t)cbc_col_groups(log) * 8), o_psum = part(kCbcUpd * 16),
                 o_list = part(kCbcFinal * 4), o_part = part((size_t)std::max(sl1 * t1, kCbcFinal * slices * ts) * 16),
                 o_out = part(64 + kMaxDim * 4 + kMaxDim * 8);
    if ((st = s.alloc(total))) return st;
    char *base = (char *)s.ptr[0];
    double *prod = (double *)(base + o_prod);
    uint32_t *perm = (uint32_t *)(base + o_perm), *list = (uint32_t *)(base + o_list);
    double2 *tw = (double2 *)(base + o_tw), *psum = (double2 *)(base + o_psum), *fpart = (double2 *)(base + o_part);
    CbcState *state = (CbcState *)(base + o_out);
    double *d_e2 = (double *)(base + o_out + 64);
    uint32_t *d_z = (uint32_t *)(base + o_out + 64 + kMaxDim * 8);

    struct {
        CbcState state;
        uint32_t pad[14];
        double e2[kMaxDim];
        uint32_t z[kMaxDim];
    } res{};
    static_assert(sizeof(res) == 64 + kMaxDim * 12, "layout of the result block");
    // the first component is the only candidate 1; its finalist list is that
    const uint32_t one_h = 1u;
    res.state.count = 1;
    if ((e = hipMemcpy(state, &res, sizeof res, hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(list, &one_h, 4, hipMemcpyHostToDevice)) != hipSuccess)
        return hip_fail(e, "cbc upload");
    hipLaunchKernelGGL(k_fill, dim3(nb), dim3(kBlock), 0, nullptr, prod, jend, 1.0);
    hipLaunchKernelGGL(k_cbc_tables, dim3((std::max<uint32_t>(N, kCbcTw) + kBlock - 1) / kBlock), dim3(kBlock), 0,
                       nullptr, tw, perm, (uint32_t)n, N, inv_n, (uint32_t)primitive_root(n));
    CbcFftArgs fa{(uint32_t)n, N, inv_n, perm, prod, tw, (double2 *)(base + o_work), (const double2 *)(base + o_spec),
                  (double *)(base + o_value), (double *)(base + o_vmin), state};
    // |p|_2 times tol bounds the error of every V: each of the three
    // transforms adds at most log2(L) 7 2^-53 of |p|_2 |B2|_2 (the transform's
    // 2-norm bound and Cauchy-Schwarz), |B2| <= 1/6 on 2N - 1 points; the
    // factor 32 covers the three and the product.  Measured errors are below
    // 2e-3 of it (n = 16381 .. 1048573).
    const double tol = 32.0 * 0x1p-53 * log * std::sqrt(2.0 * (double)N) / 6.0;
    auto exact_step = [&](uint32_t comp) {
        const bool first = comp == 0;
        const uint32_t sl = first ? sl1 : slices, ch = first ? ch1 : chs, tl = first ? t1 : ts;
        const double w = two_pi2 * gam[comp];
        const CbcArgs a{(uint32_t)n, jend, 0, ch, inv_n, w, prod, list, fpart};
        // usually one or two finalists; enough workgroups for many where a
        // lattice is a few tiles
        const uint32_t gy = first ? 1u : std::min(64u, std::max(4u, 256u / (sl * tl)));
        hipLaunchKernelGGL(k_cbc_exact, dim3(sl * tl, gy), dim3(kBlock), 0, nullptr, a, tl, (const CbcState *)state);
        hipLaunchKernelGGL(k_cbc_choose, dim3(1), dim3(1024), 0, nullptr, (const double2 *)fpart, sl * tl, (uint32_t)n,
                           inv_n, w, (const double *)prod, (const uint32_t *)list, state, comp, d_z, d_e2);
    };
    auto advance = [&](uint32_t comp, bool chosen) {
        hipLaunchKernelGGL(k_cbc_advance, dim3(kCbcUpd), dim3(kBlock), 0, nullptr, prod, (uint32_t)n, jend, inv_n,
                           chosen ? (const uint32_t *)(d_z + comp) : nullptr, chosen ? 0u : (uint32_t)z_out[comp],
                           two_pi2 * gam[comp], (const CbcState *)state, psum);
    };
    exact_step(0);
    advance(0, true);
    {
        CbcFftArgs fb = fa;  // the spectrum of B2, left where the products read it
        fb.prod = nullptr;
        fb.work = (double2 *)(base + o_spec);
        if (d > 1) cbc_fft_pass(log, fb, true);
    }
    uint32_t from = 0;  // first component not yet returned
    uint32_t over = 0;  // 1 + the component that had too many finalists (0: none)
    auto fetch = [&](uint32_t end) -> qmc_status {
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch CBC kernels");
        if ((e = hipMemcpy(&res, state, sizeof res, hipMemcpyDeviceToHost)) != hipSuccess)
            return hip_fail(e, "cbc download");
        over = res.state.overflow;
        const uint32_t done = over ? over - 1 : end;
        for (; from < done; ++from) {
            z_out[from] = res.z[from];
            e2_out[from] = res.e2[from];
        }
        return QMC_OK;
    };
    double tied = 0.0;
    auto spread = [&](uint32_t c) { return cbc_spread(gam, c, n); };
    auto unscreened = [&](uint32_t c) { return cbc_unscreened(spread(c), tied, n); };
    bool ahead = false;  // launches whose outcome the host has not waited for
    // component c by direct sums (weights near zero make too many candidates
    // alike; values that are not finite end the search there)
    auto directly = [&](uint32_t c) -> qmc_status {
        if ((st = direct(c, prod))) return st;
        const CbcState clear{0, 0};
        if (over && (e = hipMemcpy(state, &clear, sizeof clear, hipMemcpyHostToDevice)) != hipSuccess)
            return hip_fail(e, "cbc upload");
        over = 0;
        advance(c, false);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch CBC update");
        from = c + 1;
        ahead = true;
        return QMC_OK;
    };
    for (uint32_t comp = 1; comp < d || from < d;) {
        if (comp < d && !unscreened(comp)) {
            bool look = false;
            while (!look && comp < d && !unscreened(comp)) {
                cbc_fft_pass(log, fa, false);
                const CbcSelectArgs sa{(uint32_t)n, N, cbc_col_groups(log), two_pi2 * gam[comp], tol, fa.value,
                                       fa.vmin, prod, psum, perm, list, state};
                hipLaunchKernelGGL(k_cbc_select, dim3((N + kBlock - 1) / kBlock), dim3(kBlock), 0, nullptr, sa);
                exact_step(comp);
                advance(comp, true);
                look = N > kCbcFinal && spread(comp) < kTieLook * N;
                ++comp;
            }
        }
        if (from < comp) {
            if ((st = fetch(comp))) return st;
            ahead = false;
        }
        if (over) {
            comp = over - 1;
            if (comp) tied = std::max(tied, spread(comp));
            if ((st = directly(comp))) return st;
            ++comp;
        } else if (comp < d && unscreened(comp)) {
            if ((st = directly(comp))) return st;
            ++comp;
        }
    }
    if (ahead && (e = hipDeviceSynchronize()) != hipSuccess) return hip_fail(e, "cbc synchronize");
    return QMC_OK;
}
