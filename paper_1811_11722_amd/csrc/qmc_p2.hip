// P2 criterion of Korobov vectors (qmc_korobov_search in qmc.h).
//
// P2(a) = -1 + (1/n) sum_j prod_i (1 + 2 pi^2 B2({j a^i / n})) is an unshifted
// lattice sum, one per candidate multiplier a.  Unshifted points need no
// wrap in floating point, and the first coordinate of every candidate is j / n
// itself, so the search has a kernel of its own: a thread walks the exact
// indices of kP2Cand candidates at once (independent chains), forms each
// factor from the index by two FMAs,
//   1 + 2 pi^2 B2(x) = s^2 + (1 - pi^2/6),  s = sqrt(2) pi (x - 1/2),
// and shares the first one.  Per candidate and dimension that is a conversion,
// two FMAs, a multiply and three integer operations, against a multiply, an
// add and a v_fract more in the general lattice kernel; the sums are formed
// and folded the same way (chunks of kChunk points, double-double).  Bound by
// VALU issue.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "qmc_registry.hpp"
#include "qmc_runtime.hpp"

namespace qmc {

namespace {

// Candidates per thread: n = 2^24 - 3, d = 6, 64 candidates take 676 us a search
// with one, 620 with two, 605 with four and 597 with eight (1012 in the general
// lattice kernel); n = 2^20 - 3, d = 10: 113, 113, 118 and 118 us, n = 65521,
// d = 6: 46, 46, 47 and 49 us.  A search of one candidate takes one: the second
// would be a copy (n = 2^31 - 1, d = 12: 4.68 ms, 2.46 with one).
constexpr int kP2Cand = 2;

struct P2Args {
    uint32_t n, jend;       // points j < jend are summed
    uint32_t ncand, nblk;
    double inv_n;
    double kappa;           // sqrt(2) pi / n
    double c0;              // the factor's constant (p2_constant)
    const uint32_t *g;      // (groups C, D): candidates padded by repeating the last
    const uint32_t *gstep;  // (stride g_i) mod n, same layout
    double2 *partials;      // (ncand, nblk)
};

constexpr double kP2Shift = 2.221441469079183;  // sqrt(2) pi / 2

// The constant that makes the mean of s^2 + c0 over the n indices, with the
// rounded kappa and shift, equal the factor's exact mean 1 + pi^2 / (3 n^2):
// P2 is a mean of products near 1 minus 1, so a constant error of the factor
// would survive the sum while the points' own roundings average out.
double p2_constant(uint64_t n, double kappa) {
    const long double N = (long double)n, k = kappa, c = kP2Shift, pi = 3.14159265358979323846264338327950288L;
    const long double mean = k * k * (N - 1) * (2 * N - 1) / 6 - k * c * (N - 1) + c * c;
    return (double)(1 + pi * pi / (3 * N * N) - mean);
}

template <int D, int C>
__global__ __launch_bounds__(kBlock) void k_p2(const P2Args a) {
    const uint32_t c0 = blockIdx.y * C;
    const uint32_t *__restrict__ g = a.g + (size_t)c0 * D;
    const uint32_t *__restrict__ gs = a.gstep + (size_t)c0 * D;
    const uint32_t S = gridDim.x * kBlock;
    uint32_t j = blockIdx.x * kBlock + threadIdx.x;
    auto factor = [&](uint32_t idx) {
        const double s = fma_((double)idx, a.kappa, -kP2Shift);
        return fma_(s, s, a.c0);
    };
    double hi[C][1], lo[C][1];
#pragma unroll
    for (int c = 0; c < C; ++c) hi[c][0] = lo[c][0] = 0.0;
    if (j < a.jend) {
        uint32_t idx[C][D], step[C][D];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int i = 1; i < D; ++i) {
                idx[c][i] = mulmod(j, g[c * D + i], a.n, a.inv_n);
                step[c][i] = gs[c * D + i];
            }
#pragma unroll 1
        while (j < a.jend) {
            double s[C];
#pragma unroll
            for (int c = 0; c < C; ++c) s[c] = 0.0;
#pragma unroll 1
            for (int u = 0; u < kChunk && j < a.jend; ++u) {
                const double first = factor(j);  // g_0 = 1 and j < n
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    double prod = first;
#pragma unroll
                    for (int i = 1; i < D; ++i) {
                        prod *= factor(idx[c][i]);
                        const uint32_t t = idx[c][i] + step[c][i];  // < 2n <= 2^32
                        idx[c][i] = min(t, t - a.n);                // t - n wraps above t when t < n
                    }
                    s[c] += prod;
                }
                j += S;
            }
#pragma unroll
            for (int c = 0; c < C; ++c) dd_accumulate(hi[c][0], lo[c][0], s[c]);
        }
    }
    __shared__ dd red[kBlock / kWave][C];
    const dd r = block_reduce<C, 1>(hi, lo, red);
    if (threadIdx.x < (uint32_t)C && c0 + threadIdx.x < a.ncand)
        a.partials[(size_t)(c0 + threadIdx.x) * a.nblk + blockIdx.x] = make_double2(r.hi, r.lo);
}

template <int D>
hipError_t launch_p2_from(uint32_t d, uint32_t per_thread, const P2Args &a, dim3 grid, hipStream_t s) {
    if constexpr (D > (int)kMaxDim) {
        return hipErrorInvalidValue;
    } else {
        if (d != (uint32_t)D) return launch_p2_from<D + 1>(d, per_thread, a, grid, s);
        if (per_thread == 1) hipLaunchKernelGGL((k_p2<D, 1>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((k_p2<D, kP2Cand>), grid, dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
}

}  // namespace
}  // namespace qmc

using namespace qmc;

extern "C" qmc_status qmc_korobov_search(uint64_t n, uint32_t d, const uint64_t *cand, uint32_t ncand,
                                         uint64_t *a_best, double *p2_best, double *p2_all) {
    if (!cand || !a_best || !p2_best) return fail(QMC_EINVAL, "null argument");
    if (ncand == 0) return fail(QMC_EINVAL, "ncand must be >= 1");
    if (ncand > 4096) return fail(QMC_EUNSUPPORTED, "ncand > 4096");
    if (d == 0) return fail(QMC_EINVAL, "d must be >= 1");
    if (d > kMaxDim) return fail(QMC_EUNSUPPORTED, "d > %u", kMaxDim);
    if (n < 2) return fail(QMC_EINVAL, "n must be >= 2");
    if (n > (1ull << 31)) return fail(QMC_EUNSUPPORTED, "n > 2^31");
    for (uint32_t c = 0; c < ncand; ++c)
        if (cand[c] % n == 0) return fail(QMC_EINVAL, "candidate %u is 0 mod n", c);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    // The point n - j is the mirror 1 - x of the point j and B2(1 - x) =
    // B2(x), so the sum S over all points is 2 sum_{j <= n/2} - term(0) -
    // [n even] term(n/2), term(0) = (1 + pi^2/3)^d.  For even n and odd
    // candidates every g_i is odd and the point n/2 is (1/2, ..., 1/2) for
    // all of them; an even candidate puts 0 in some coordinates there, and
    // then all n points are summed.  Both terms are formed as the kernel
    // forms them, multiplied up in order.
    bool half = true;
    if ((n & 1) == 0)
        for (uint32_t c = 0; c < ncand; ++c) half = half && (cand[c] % n) % 2 == 1;
    const uint32_t per_thread = ncand == 1 ? 1 : kP2Cand;
    const uint32_t groups = (ncand + per_thread - 1) / per_thread, padded = groups * per_thread;
    const uint32_t bx = grid_x((uint32_t)n, groups, dev, 8);
    std::vector<uint32_t> tab(2 * (size_t)padded * d);  // g, then gstep
    uint32_t *g = tab.data(), *gs = g + (size_t)padded * d;
    for (uint32_t c = 0; c < padded; ++c) {
        const uint64_t a = cand[std::min(c, ncand - 1)] % n;
        uint64_t v = 1 % n;
        for (uint32_t i = 0; i < d; ++i) {
            g[(size_t)c * d + i] = (uint32_t)v;
            v = (v * a) % n;
        }
        gstep_for(&g[(size_t)c * d], d, (uint32_t)n, (uint64_t)bx * kBlock, &gs[(size_t)c * d]);
    }
    // one allocation: block pairs, per-candidate values, results, tables
    const size_t o_q = (size_t)ncand * bx * sizeof(double2), o_res = o_q + (size_t)ncand * 8,
                 o_tab = o_res + (size_t)ncand * 32;
    DeviceScratch s;
    qmc_status st = s.alloc(o_tab + tab.size() * 4);
    if (st) return st;
    char *base = (char *)s.ptr[0];
    if ((e = hipMemcpy(base + o_tab, tab.data(), tab.size() * 4, hipMemcpyHostToDevice)) != hipSuccess)
        return hip_fail(e, "search upload");
    P2Args a{};
    a.n = (uint32_t)n;
    a.jend = half ? (uint32_t)(n / 2 + 1) : (uint32_t)n;
    a.ncand = ncand;
    a.nblk = bx;
    a.inv_n = 1.0 / (double)n;
    a.kappa = 2.0 * kP2Shift / (double)n;
    a.c0 = p2_constant(n, a.kappa);
    a.g = (const uint32_t *)(base + o_tab);
    a.gstep = a.g + (size_t)padded * d;
    a.partials = (double2 *)base;
    double t0 = 0.0;
    if (half) {
        auto factor = [&](double idx) {
            const double v = std::fma(idx, a.kappa, -kP2Shift);
            return std::fma(v, v, a.c0);
        };
        auto power = [d](double q) {
            double t = q;
            for (uint32_t i = 1; i < d; ++i) t *= q;
            return t;
        };
        t0 = power(factor(0.0));
        if ((n & 1) == 0) t0 += power(factor((double)(n / 2)));  // both self-mirrored terms
    }
    if ((e = launch_p2_from<1>(d, per_thread, a, dim3(bx, groups), nullptr)) != hipSuccess) return hip_fail(e, "launch P2 kernel");
    FinalizeArgs f{};
    f.partials = a.partials;
    f.nblk = bx;
    f.m = 1;
    f.np = 1;
    f.n = (double)n;
    // q = (S - n) / n = ((sum - (n + t0) / 2) 2) / n, t0 the self-mirrored terms
    f.scale = half ? 2.0 : 1.0;
    f.sub = half ? ((double)n + t0) / 2.0 : (double)n;
    f.q = (double *)(base + o_q);
    f.res = (double *)(base + o_res);
    if ((e = launch_finalize(f, ncand, nullptr)) != hipSuccess) return hip_fail(e, "launch finalize");
    std::vector<double> p2(ncand);
    if ((e = hipMemcpy(p2.data(), f.q, ncand * 8, hipMemcpyDeviceToHost)) != hipSuccess)
        return hip_fail(e, "search download");
    uint64_t best_a = 0;
    double best = INFINITY;
    for (uint32_t c = 0; c < ncand; ++c) {
        if (p2_all) p2_all[c] = p2[c];
        if (p2[c] < best || (p2[c] == best && cand[c] < best_a)) {
            best = p2[c];
            best_a = cand[c];
        }
    }
    if (!std::isfinite(best)) return fail(QMC_ENONFINITE, "P2 not finite");
    *a_best = best_a;
    *p2_best = best;
    return QMC_OK;
}
