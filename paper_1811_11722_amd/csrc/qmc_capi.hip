// Host runtime and C ABI of the lattice estimator (declarations in qmc.h).
//
// A plan holds the rule of eq. (2) of arXiv:1811.11722 -- d, n, g, m, the m
// shifts and the periodising transform -- resident in device memory.  Each
// qmc_integrate call packs the integrand parameters into a blob (uploaded
// only when it changed), launches the lattice kernel and the finalize kernel
// on the plan's stream, which writes the m per-shift values and the
// (mean, error) of eqs. (2)-(3) to the plan's pinned memory: one small
// host->device copy at most per estimate and no copy back.
#include "qmc_runtime.hpp"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <numeric>

namespace qmc {

// ------------------------------------------------------------------ errors
static thread_local std::string g_last_error;

qmc_status fail(qmc_status s, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return s;
}

qmc_status hip_fail(hipError_t e, const char *what) {
    return fail(QMC_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

int device_cu_count(int dev) {
    static std::map<int, int> cache;
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    int cu = 0;
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0)
        cu = 256;
    cache[dev] = cu;
    return cu;
}

// ------------------------------------------------------- parameter packing
static inline double bits(uint64_t v) {
    double d;
    std::memcpy(&d, &v, sizeof d);
    return d;
}

static bool finite_all(const double *p, size_t n) {
    for (size_t i = 0; i < n; ++i)
        if (!std::isfinite(p[i])) return false;
    return true;
}

// factor-list code of one monomial: count in bits 0..3, then 5 bits per factor
static qmc_status monomial_code(const uint8_t *e, uint32_t d, uint64_t &code) {
    uint64_t c = 0;
    uint32_t cnt = 0;
    for (uint32_t i = 0; i < d; ++i) {
        if (e[i] > 2) return fail(QMC_EINVAL, "exponent %u > 2 in variable %u", (unsigned)e[i], i);
        for (uint32_t r = 0; r < e[i]; ++r) {
            if (cnt >= 12) return fail(QMC_EUNSUPPORTED, "monomial of total degree > 12");
            c |= (uint64_t)i << (4 + 5 * cnt);
            ++cnt;
        }
    }
    code = c | cnt;
    return QMC_OK;
}

qmc_status pack_params(int family, uint32_t d, const void *params, Packed &pk) {
    const uint32_t D = d;
    std::vector<double> keep = std::move(pk.blob);  // its storage
    pk = Packed{};
    pk.blob = std::move(keep);
    pk.blob.clear();
    pk.key_family = family;
    switch (family) {
    case QMC_F_CONST: {
        if (!params) return fail(QMC_EINVAL, "QMC_F_CONST needs qmc_const_params");
        const auto *p = static_cast<const qmc_const_params *>(params);
        if (!std::isfinite(p->c)) return fail(QMC_EINVAL, "constant is not finite");
        pk.blob = {p->c};
        break;
    }
    case QMC_F_P2KERNEL:
        pk.blob = {0.0};
        break;
    case QMC_F_TRIG: {
        if (!params) return fail(QMC_EINVAL, "QMC_F_TRIG needs qmc_trig_params");
        const auto *p = static_cast<const qmc_trig_params *>(params);
        if (p->n_terms > 4096) return fail(QMC_EUNSUPPORTED, "more than 4096 trigonometric terms");
        if (p->n_terms && (!p->h || !p->c || !p->phi)) return fail(QMC_EINVAL, "null trig arrays");
        if (!std::isfinite(p->c0)) return fail(QMC_EINVAL, "c0 is not finite");
        pk.blob.push_back(bits(p->n_terms));
        pk.blob.push_back(p->c0);
        for (uint32_t t = 0; t < p->n_terms; ++t) {
            if (!std::isfinite(p->c[t]) || !std::isfinite(p->phi[t]))
                return fail(QMC_EINVAL, "trig coefficient %u is not finite", t);
            pk.blob.push_back(p->c[t]);
            pk.blob.push_back(p->phi[t] / (2.0 * M_PI));
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back((double)p->h[(size_t)t * d + i]);
        }
        break;
    }
    case QMC_F_GENZ_PRODUCT_PEAK:
    case QMC_F_GENZ_OSCILLATORY:
    case QMC_F_GENZ_GAUSSIAN:
    case QMC_F_GENZ_CONTINUOUS:
    case QMC_F_GENZ_CORNER_PEAK: {
        if (!params) return fail(QMC_EINVAL, "Genz family needs qmc_genz_params");
        const auto *p = static_cast<const qmc_genz_params *>(params);
        if (!p->a || !p->u) return fail(QMC_EINVAL, "null Genz arrays");
        if (!finite_all(p->a, d) || !finite_all(p->u, d)) return fail(QMC_EINVAL, "Genz parameter not finite");
        if (family == QMC_F_GENZ_PRODUCT_PEAK) {
            for (uint32_t i = 0; i < d; ++i)
                if (p->a[i] == 0.0) return fail(QMC_EINVAL, "product peak needs a_i != 0");
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(1.0 / (p->a[i] * p->a[i]));
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->u[i]);
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(0.5 - p->u[i]);
            // tile flag: one reciprocal may serve a thread's shifts if every
            // denominator prod_i q_i, a^-2 <= q_i <= a^-2 + max(u^2, (1-u)^2),
            // lies within 2^-62 .. 2^62 (products of up to 16 of them then stay
            // within 2^-1000 .. 2^1000)
            double lg_lo = 0.0, lg_hi = 0.0;
            for (uint32_t i = 0; i < d; ++i) {
                const double a2 = 1.0 / (p->a[i] * p->a[i]);
                const double s2 = std::max(p->u[i] * p->u[i], (1.0 - p->u[i]) * (1.0 - p->u[i]));
                lg_lo += std::log2(a2);
                lg_hi += std::log2(a2 + s2);
            }
            pk.blob.push_back(std::isfinite(lg_lo) && std::isfinite(lg_hi) && lg_lo >= -62.0 && lg_hi <= 62.0 ? 1.0
                                                                                                                : 0.0);
        } else if (family == QMC_F_GENZ_OSCILLATORY) {
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->a[i]);
            pk.blob.push_back(2.0 * M_PI * p->u[0]);
        } else if (family == QMC_F_GENZ_GAUSSIAN) {
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->a[i] * p->a[i]);
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->u[i]);
        } else if (family == QMC_F_GENZ_CONTINUOUS) {
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->a[i]);
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->u[i]);
        } else {
            for (uint32_t i = 0; i < D; ++i) pk.blob.push_back(p->a[i]);
        }
        break;
    }
    case QMC_F_SECTOR: {
        if (!params) return fail(QMC_EINVAL, "QMC_F_SECTOR needs qmc_sector_params");
        const auto *p = static_cast<const qmc_sector_params *>(params);
        if (p->n_u == 0 || p->n_f == 0) return fail(QMC_EINVAL, "n_u and n_f must be >= 1");
        if (p->n_u > 4096 || p->n_f > 4096) return fail(QMC_EUNSUPPORTED, "more than 4096 monomials");
        if (!p->coef_u || !p->exp_u || !p->coef_f || !p->exp_f || !p->nu)
            return fail(QMC_EINVAL, "null sector arrays");
        if (!finite_all(p->coef_u, p->n_u) || !finite_all(p->coef_f, p->n_f))
            return fail(QMC_EINVAL, "polynomial coefficient not finite");
        if (!std::isfinite(p->pow_u) || !std::isfinite(p->pow_f)) return fail(QMC_EINVAL, "power not finite");
        const bool cplx = p->is_complex != 0;
        if (cplx && (!std::isfinite(p->delta_im))) return fail(QMC_EINVAL, "delta_im not finite");
        // the phase pow_f * arg(F - i delta) must stay inside the exact range
        // of the device sine and cosine (|x| < 2^19)
        if (cplx && std::fabs(p->pow_f) > 1.0e5) return fail(QMC_EUNSUPPORTED, "|pow_f| > 1e5 for a complex sector");
        uint64_t nucode = 0;
        for (uint32_t i = 0; i < d; ++i) {
            if (p->nu[i] > 2) return fail(QMC_EINVAL, "nu_%u = %u > 2", i, (unsigned)p->nu[i]);
            nucode |= (uint64_t)p->nu[i] << (2 * i);
        }
        qmc_status st = QMC_OK;
        uint32_t flags = (cplx ? 1u : 0u) | (p->pow_u == -2.0 ? 2u : 0u);
        pk.blob = {bits(p->n_u), bits(p->n_f), bits(flags), p->pow_u, p->pow_f, cplx ? p->delta_im : 0.0,
                   bits(nucode)};
        // terms are stored in the order the specialised code reads them (the
        // polynomial is the same sum in any order)
        std::vector<uint64_t> cu(p->n_u), cf(p->n_f);
        for (uint32_t t = 0; t < p->n_u; ++t)
            if ((st = monomial_code(p->exp_u + (size_t)t * d, d, cu[t]))) return st;
        for (uint32_t t = 0; t < p->n_f; ++t)
            if ((st = monomial_code(p->exp_f + (size_t)t * d, d, cf[t]))) return st;
        const std::vector<uint32_t> ou = horner_term_order(cu, d), of = horner_term_order(cf, d);
        for (uint32_t t : ou) pk.blob.push_back(p->coef_u[t]);
        for (uint32_t t : ou) pk.blob.push_back(bits(cu[t]));
        for (uint32_t t : of) pk.blob.push_back(p->coef_f[t]);
        for (uint32_t t : of) pk.blob.push_back(bits(cf[t]));
        if (cplx) {
            pk.np = 2;
            pk.key_family = kFamSectorComplex;
            pk.cplx = true;
        }
        if (p->n_orders >= 2) {
            if (p->n_orders > kSectorMaxOrders)
                return fail(QMC_EUNSUPPORTED, "n_orders = %u > %u", p->n_orders, kSectorMaxOrders);
            if (!std::isfinite(p->eps_u) || !std::isfinite(p->eps_f)) return fail(QMC_EINVAL, "eps not finite");
            flags |= kSectorOrders;
            pk.blob[2] = bits(flags);
            pk.blob.push_back(p->eps_u);
            pk.blob.push_back(p->eps_f);
            pk.blob.push_back(bits(p->n_orders));
            pk.orders = p->n_orders;
            pk.np *= p->n_orders;
        }
        if (p->deform_lambda != 0.0) {
            if (!std::isfinite(p->deform_lambda)) return fail(QMC_EINVAL, "deform_lambda not finite");
            if (std::fabs(p->pow_f) > 1.0e5 || std::fabs(p->pow_u) > 1.0e5)
                return fail(QMC_EUNSUPPORTED, "|pow_u| or |pow_f| > 1e5 for a deformed sector");
            flags |= kSectorComplex | kSectorDeform;
            pk.blob[2] = bits(flags);
            pk.blob.push_back(p->deform_lambda);
            std::vector<uint64_t> stored;
            for (uint32_t t : of) stored.push_back(cf[t]);
            for (const auto &e : derivative_sources(stored, d)) pk.blob.push_back(e.second * p->coef_f[of[e.first]]);
            pk.deform = true;
            pk.cplx = true;
            pk.key_family = kFamSectorComplex;
            // Re, Im per order, then the count of points on the wrong side
            pk.np = 2 * (p->n_orders >= 2 ? p->n_orders : 1u) + 1;
            pk.crossing = true;
        }
        break;
    }
    default:
        return fail(QMC_EINVAL, "unknown family %d", family);
    }
    return QMC_OK;
}

// Calls fn(pointer, bytes) for every value of the parameters, in a fixed
// order, until it returns false; false too for parameters that pack_params
// would refuse to read.
template <class Fn>
static bool raw_walk(int family, uint32_t d, const void *params, Fn &&fn) {
    auto one = [&](const auto &v) { return fn(&v, sizeof v); };
    auto many = [&](const auto *v, size_t n) { return n == 0 || (v && fn(v, n * sizeof *v)); };
    if (family == QMC_F_P2KERNEL) return true;
    if (!params) return false;
    if (family == QMC_F_CONST) return one(static_cast<const qmc_const_params *>(params)->c);
    if (family == QMC_F_TRIG) {
        const auto &p = *static_cast<const qmc_trig_params *>(params);
        return p.n_terms <= 4096 && one(p.n_terms) && one(p.c0) && many(p.h, (size_t)p.n_terms * d) &&
               many(p.c, p.n_terms) && many(p.phi, p.n_terms);
    }
    if (family == QMC_F_SECTOR) {
        const auto &p = *static_cast<const qmc_sector_params *>(params);
        return p.n_u <= 4096 && p.n_f <= 4096 && one(p.n_u) && one(p.n_f) && many(p.coef_u, p.n_u) &&
               many(p.exp_u, (size_t)p.n_u * d) && many(p.coef_f, p.n_f) && many(p.exp_f, (size_t)p.n_f * d) &&
               many(p.nu, d) && one(p.pow_u) && one(p.pow_f) && one(p.delta_im) && one(p.is_complex) &&
               one(p.n_orders) && one(p.eps_u) && one(p.eps_f) && one(p.deform_lambda);
    }
    if (family < QMC_F_GENZ_PRODUCT_PEAK || family > QMC_F_GENZ_CORNER_PEAK) return false;
    const auto &p = *static_cast<const qmc_genz_params *>(params);
    return many(p.a, d) && many(p.u, d);
}

bool raw_match(const RawParams &raw, size_t &at, int family, uint32_t d, const void *params) {
    return raw.family == family && raw_walk(family, d, params, [&](const void *v, size_t n) {
        if (raw.bytes.size() - at < n || std::memcmp(raw.bytes.data() + at, v, n) != 0) return false;
        at += n;
        return true;
    });
}

bool raw_same(const RawParams &raw, int family, uint32_t d, const void *params) {
    size_t at = 0;
    return raw_match(raw, at, family, d, params) && at == raw.bytes.size();
}

bool raw_append(RawParams &raw, int family, uint32_t d, const void *params) {
    size_t size = raw.bytes.size();
    if (!raw_walk(family, d, params, [&](const void *, size_t n) { return size += n, true; })) {
        raw.family = -1;
        return false;
    }
    size_t at = raw.bytes.size();
    raw.bytes.resize(size);
    raw_walk(family, d, params, [&](const void *v, size_t n) {
        std::memcpy(raw.bytes.data() + at, v, n);
        at += n;
        return true;
    });
    raw.family = family;
    return true;
}

// The packed integrand of a plan's call: the last one when the caller's values
// are the same bytes (packing a d = 6 sector of 42 monomials takes 1.5 us and
// building its kernel's key 3 us, of a call of 22), packed anew otherwise (with
// the upload and its wait, a call with new coefficients takes 38 us).
qmc_status plan_pack(qmc_plan_s *p, int family, const void *params, const Packed *&pk) {
    pk = &p->last_pk;
    if (raw_same(p->last_raw, family, p->d, params)) return QMC_OK;
    p->last_raw.family = -1;
    p->last_raw.bytes.clear();
    p->last_fn_T = 0;
    const qmc_status st = pack_params(family, p->d, params, p->last_pk);
    if (st) return st;
    raw_append(p->last_raw, family, p->d, params);
    return QMC_OK;
}

// The table-driven kernels' form of a sector blob (qmc_integrands.hpp):
// coefficients of degree up to three in their Horner slots (d <= kTabMaxD), the
// other terms and repeated monomials as coded factor lists.  Formed in `out`;
// other families' blobs are returned as they are.
const std::vector<double> &table_blob(const Packed &pk, uint32_t d, std::vector<double> &out) {
    if (pk.key_family != QMC_F_SECTOR && pk.key_family != kFamSectorComplex) return pk.blob;
    const std::vector<double> &b = pk.blob;
    auto word = [&](size_t i) {
        uint64_t v;
        std::memcpy(&v, &b[i], sizeof v);
        return v;
    };
    const int D = (int)d, size = tab_words(D);
    out.assign(kSectorHeader + 2 * (size_t)size, 0.0);
    std::vector<double> lists;
    std::copy(b.begin(), b.begin() + kSectorHeader, out.begin());
    size_t at = kSectorHeader;
    for (int w = 0; w < 2; ++w) {
        const size_t n = word(w);
        double *tab = out.data() + kSectorHeader + (size_t)w * size;
        std::vector<uint32_t> mask(size, 0u);
        std::vector<char> used(size, 0);
        std::vector<double> coef, code;
        for (size_t t = 0; t < n; ++t) {
            const double c = b[at + t];
            const uint64_t m = word(at + n + t);
            const uint32_t cnt = (uint32_t)(m & 15u);
            // factors ascend (monomial_code)
            const int v0 = (int)((m >> 4) & 31u), v1 = (int)((m >> 9) & 31u), v2 = (int)((m >> 14) & 31u);
            if (D > kTabMaxD) {
                coef.push_back(c);
                code.push_back(bits(m));
                continue;
            }
            const int slot = cnt == 0   ? 0
                             : cnt == 1 ? tab_a_off(D, v0)
                             : cnt == 2 ? tab_pair_off(D, v0, v1)
                                        : tab_pair_off(D, v0, v1) + 2 + v2 - v1;
            if (cnt > 3 || used[slot]) {
                coef.push_back(c);
                code.push_back(bits(m));
                continue;
            }
            used[slot] = 1;
            tab[slot] = c;
            if (cnt >= 1) mask[tab_a_off(D, v0) + 1] |= kTabPresent;
            if (cnt >= 2) mask[tab_a_off(D, v0) + 1] |= 1u << v1;
            if (cnt == 3) mask[tab_pair_off(D, v0, v1) + 1] |= 1u << v2;
        }
        for (int i = 0; i < size; ++i)
            if (mask[i]) tab[i] = bits(mask[i]);
        out[w] = bits(coef.size());
        lists.insert(lists.end(), coef.begin(), coef.end());
        lists.insert(lists.end(), code.begin(), code.end());
        at += 2 * n;
    }
    out.insert(out.end(), lists.begin(), lists.end());
    return out;
}

double transform_scale(const qmc_transform &t, uint32_t d) {
    if (t.kind == QMC_T_SIDI) {
        // 1 / T_m per dimension, T_m = int_0^1 sin^m(pi x) dx
        const int m = t.alpha, p = m / 2;
        double tm;
        if (m % 2 == 0) {
            tm = 1.0;  // binom(2p, p) / 4^p
            for (int k = 1; k <= p; ++k) tm *= (double)(p + k) / (4.0 * k);
        } else {
            double p1 = 0.0, b = 1.0;  // sum_k binom(p, k) (-1)^k / (2k + 1)
            for (int k = 0; k <= p; ++k) {
                p1 += ((k & 1) ? -b : b) / (2 * k + 1);
                b = b * (p - k) / (k + 1);
            }
            tm = 2.0 * p1 / 3.141592653589793;
        }
        return std::pow(1.0 / tm, (double)d);
    }
    if (t.kind != QMC_T_KOROBOV) return 1.0;
    double c = 1.0;  // (2a+1)! / (a!)^2
    for (int k = t.alpha + 1; k <= 2 * t.alpha + 1; ++k) c *= k;
    for (int k = 2; k <= t.alpha; ++k) c /= k;
    return std::pow(c, (double)d);
}

// ------------------------------------------------------------ kernel choice
static const int kTChoices[] = {8, 4, 2, 1};

LatticeLaunch find_kernel(int key_family, const qmc_transform &t, uint32_t d, uint32_t want_T,
                          uint32_t &T_out) {
    auto &reg = lattice_registry();
    const int alpha = (t.kind == QMC_T_KOROBOV || t.kind == QMC_T_SIDI) ? t.alpha : 0;
    if (want_T) {
        auto it = reg.find(KernelKey{key_family, t.kind, alpha, (int)d, (int)want_T});
        if (it != reg.end()) {
            T_out = want_T;
            return it->second;
        }
    }
    for (int T : kTChoices) {
        auto it = reg.find(KernelKey{key_family, t.kind, alpha, (int)d, T});
        if (it != reg.end()) {
            T_out = (uint32_t)T;
            return it->second;
        }
    }
    return nullptr;
}

uint32_t default_tile(int key_family) {
    switch (key_family) {
    case QMC_F_GENZ_PRODUCT_PEAK: return 4;
    case QMC_F_SECTOR: return 2;
    case kFamSectorComplex: return 1;
    case QMC_F_P2KERNEL: return 1;
    default: return 4;
    }
}

// Workgroups along the points: about blocks_per_cu (default 8) per CU over
// all shift tiles, and fewer at small n, where a thread's start (exact products
// of 64 bits) and the block reduction weigh as much as its walk: at least 32
// points per thread, down to 4 while there are fewer than two workgroups per CU
// and to one while some CU has none.  d = 6 sector, m = 32, kernel time: n = 2^20 - 3
// 150 us with 32 points per thread, 163 with 8; n = 131071 26.6 us with 8 (two
// workgroups per CU), 29.3 with 4, 28.5 with 16; n = 16381, m = 16 7.0 us with
// one, 11.1 with four.
// Between one and eight workgroups per CU that count is then raised to a whole
// number per CU: with 2.1 of them on average some CUs have three and the rest
// wait for those.  Gaussian in d = 12 under Korobov 3, n = 1.1e6, m = 16: 2.1 per
// CU 164 us, 3 per CU 125, 8 per CU 135; d = 8 sector, m = 28, n = 6e5: 154 (2.0 and
// a bit), 112 and 137 us.  The nearest whole number instead: 128 and 111 us.
// min_points: 32 by default; 4 where the caller asked for a number of workgroups
// per CU (a plan's launch configuration, the autotuner) and for kernels that need
// more waves (the control-variate residual, see there).
uint32_t grid_x(uint32_t n, uint32_t tiles_total, int dev, uint32_t blocks_per_cu, uint32_t min_points) {
    const uint64_t cus = (uint64_t)device_cu_count(dev), tiles = std::max<uint32_t>(1, tiles_total);
    auto groups = [n](uint64_t per) { return (n + kBlock * per - 1) / (kBlock * per); };
    const uint64_t cap = std::max({groups(min_points), std::min(groups(4), 2 * cus / tiles), std::min(groups(1), cus / tiles)});
    const uint64_t bx = std::max<uint64_t>(1, cus * (blocks_per_cu ? blocks_per_cu : 8) / tiles);
    if (bx <= cap) return (uint32_t)bx;
    const uint64_t whole = (cap * tiles + cus - 1) / cus * cus / tiles;  // at least cap
    return (uint32_t)std::max<uint64_t>(1, cap * tiles > cus ? std::min(bx, whole) : cap);
}

void gstep_for(const uint32_t *g, uint32_t d, uint32_t n, uint64_t S, uint32_t *out) {
    const uint64_t s = S % n;
    for (uint32_t i = 0; i < d; ++i) out[i] = (uint32_t)((s * (uint64_t)g[i]) % n);
}

// shift tables on the device hold whole tiles of up to kMaxTile rows; rows
// past m repeat the last shift (their sums are never read)
uint32_t padded_rows(uint32_t m) { return (m + kMaxTile - 1) / kMaxTile * kMaxTile; }

// The baker's transform reads its points moved by 1/2 and unwrapped
// (TrBaker): the device table holds {Delta + 1/2} - 1 for it, so
// the move costs nothing per point.
std::vector<double> padded_shifts(const std::vector<double> &sh, uint32_t m, uint32_t d, uint32_t rows,
                                  const qmc_transform &tr) {
    const bool half = tr.kind == QMC_T_BAKER;
    std::vector<double> out((size_t)rows * d);
    for (uint32_t r = 0; r < rows; ++r)
        for (uint32_t i = 0; i < d; ++i) {
            const double v = sh[(size_t)std::min(r, m - 1) * d + i];
            out[(size_t)r * d + i] = !half ? v : (v < 0.5 ? v - 0.5 : v - 1.5);
        }
    return out;
}

// --------------------------------------------------------------- plan ops
qmc_status plan_upload_params(qmc_plan_s *p, const std::vector<double> &blob) {
    if (blob.size() > p->params_cap) {
        if (p->d_params) hipFree(p->d_params);
        p->d_params = nullptr;
        p->params_cap = 0;
        hipError_t e = hipMalloc(&p->d_params, blob.size() * sizeof(double));
        if (e != hipSuccess) return fail(QMC_ENOMEM, "hipMalloc params: %s", hipGetErrorString(e));
        p->params_cap = blob.size();
        p->last_blob.clear();
    }
    if (blob != p->last_blob) {
        hipError_t e = hipMemcpyAsync(p->d_params, blob.data(), blob.size() * sizeof(double),
                                      hipMemcpyHostToDevice, p->stream);
        if (e != hipSuccess) return hip_fail(e, "upload params");
        e = hipStreamSynchronize(p->stream);
        if (e != hipSuccess) return hip_fail(e, "upload params");
        p->last_blob = blob;
    }
    return QMC_OK;
}

qmc_status ensure_buffer(void **ptr, size_t &cap, size_t bytes, const char *what) {
    if (bytes <= cap) return QMC_OK;
    if (*ptr) hipFree(*ptr);
    *ptr = nullptr;
    cap = 0;
    hipError_t e = hipMalloc(ptr, bytes);
    if (e != hipSuccess) return fail(QMC_ENOMEM, "hipMalloc %s (%zu bytes): %s", what, bytes, hipGetErrorString(e));
    cap = bytes;
    return QMC_OK;
}

qmc_status plan_set_gstep(qmc_plan_s *p, uint32_t S) {
    if (S == p->cur_S) return QMC_OK;
    std::vector<uint32_t> gs(p->d);
    gstep_for(p->g.data(), p->d, p->n, S, gs.data());
    hipError_t e = hipMemcpyAsync(p->d_gstep, gs.data(), p->d * sizeof(uint32_t), hipMemcpyHostToDevice, p->stream);
    if (e != hipSuccess) return hip_fail(e, "upload gstep");
    e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) return hip_fail(e, "upload gstep");
    p->cur_S = S;
    return QMC_OK;
}

// Enqueue the lattice kernel (a registry launcher or a specialised module
// function) and the finalize kernel of one estimate.
static qmc_status plan_launch(qmc_plan_s *p, const Packed &pk, LatticeLaunch fn, hipFunction_t jfn, uint32_t T,
                              uint32_t bpc, uint32_t min_points) {
    if (p->m * pk.np > kMaxRows) return fail(QMC_EUNSUPPORTED, "m * parts > %u", kMaxRows);
    std::vector<double> table;
    qmc_status st = plan_upload_params(p, jfn ? pk.blob : table_blob(pk, p->d, table));
    if (st) return st;
    const uint32_t tiles = (p->m + T - 1) / T;
    const uint32_t bx = grid_x(p->n, tiles, p->device, bpc, min_points);
    if ((st = plan_set_gstep(p, bx * kBlock))) return st;
    const size_t pbytes = (size_t)p->m * pk.np * bx * sizeof(double2);
    if ((st = ensure_buffer((void **)&p->d_partials, p->partials_cap, pbytes, "partials"))) return st;

    LatticeArgs a{};
    a.n = p->n;
    a.d = p->d;
    a.m = p->m;
    a.tiles = tiles;
    a.inv_n = p->inv_n;
    a.g = p->d_g;
    a.gstep = p->d_gstep;
    a.shifts = p->d_shifts;
    a.params = p->d_params;
    a.g_stride = a.shift_stride = a.param_stride = 0;
    a.np = pk.np;
    a.partials = p->d_partials;
    if (p->timing) hipEventRecord(p->ev0, p->stream);
    hipError_t e = jfn ? jit_launch(jfn, a, dim3(bx, tiles), p->stream) : fn(a, dim3(bx, tiles), p->stream);
    if (e != hipSuccess) return hip_fail(e, "launch lattice kernel");
    if (p->timing) hipEventRecord(p->ev1, p->stream);

    FinalizeArgs f{};
    f.partials = p->d_partials;
    f.nblk = bx;
    f.m = p->m;
    f.np = pk.np;
    f.n = (double)p->n;
    f.scale = transform_scale(p->tr, p->d);
    f.sub = 0.0;
    f.q = p->h_out;
    f.res = p->h_out + out_res_offset(p->m);
    e = launch_finalize(f, 1, p->stream);
    if (e != hipSuccess) return hip_fail(e, "launch finalize kernel");
    p->last_T = T;
    p->last_bx = bx;
    p->last_jit = jfn != nullptr;
    return QMC_OK;
}

qmc_status plan_enqueue_fn(qmc_plan_s *p, const Packed &pk, hipFunction_t jfn, uint32_t T, uint32_t min_points) {
    return plan_launch(p, pk, nullptr, jfn, T, p->launch.blocks_per_cu, min_points);
}

// Shifts per thread of the specialised kernels: four for real sectors of up to
// eight dimensions and for real expansion orders up to six, two for the others,
// one with a deformation, whose point carries the Jacobian's triangle.  Four
// against two, kernel us at n = 2^22 - 3, m = 32 (medians, the two in turn):
//                  d = 6        7           8           9           10
// baker            477 / 507   521 / 544   523 / 557   552 / 589   578 / 608
// Korobov 2        588 / 628   673 / 702   681 / 718   740 / 775   948 / 834
// orders, baker    568 / 585   620 / 643   622 / 647   653 / 675   745 / 708
// orders, Kor. 2   687 / 720   765 / 784   855 / 821   842 / 878   971 / 936
// complex                                                          883 / 881
// So four would do at d = 9 too and, without a weight, at d = 10 (5 to 6 %); past
// that it depends on the map.  The line stays at eight, the default that
// callers and its test know.
uint32_t jit_tile(const Packed &pk, uint32_t d) {
    if (pk.deform) return 1;
    return !pk.cplx && d <= (pk.orders < 2 ? 8u : 6u) ? 4 : 2;
}

qmc_status plan_enqueue(qmc_plan_s *p, const Packed &pk, uint32_t want_T, uint32_t bpc) {
    uint32_t T = 0;
    LatticeLaunch fn = nullptr;
    hipFunction_t jfn = nullptr;
    const bool sector = pk.key_family == QMC_F_SECTOR || pk.key_family == kFamSectorComplex;
    if (sector && p->jit_mode != 0) {
        T = want_T ? want_T : jit_tile(pk, p->d);
        std::string err;
        if (&pk == &p->last_pk && p->last_fn_T == T && T)
            jfn = p->last_fn;
        else
            jfn = jit_kernel(pk.blob, p->d, p->tr, T, pk.cplx, p->device, err);
        if (&pk == &p->last_pk && jfn) {
            p->last_fn = jfn;
            p->last_fn_T = T;
        }
        if (!jfn && (p->jit_mode == 2 || pk.orders >= 2 || pk.deform))
            return fail(QMC_EUNSUPPORTED, "specialised sector kernel: %s", err.c_str());
    }
    if (!jfn && pk.orders >= 2) return fail(QMC_EUNSUPPORTED, "expansion orders need the specialised kernel (jit mode 1 or 2)");
    if (!jfn && pk.deform) return fail(QMC_EUNSUPPORTED, "contour deformation needs the specialised kernel (jit mode 1 or 2)");
    if (!jfn) {
        fn = find_kernel(pk.key_family, p->tr, p->d, want_T ? want_T : default_tile(pk.key_family), T);
        if (!fn)
            return fail(QMC_EUNSUPPORTED, "no kernel for family %d, transform %d/%d, d = %u", pk.key_family,
                        p->tr.kind, p->tr.alpha, p->d);
    }
    const uint32_t min_points = bpc ? 4 : 32;  // a number asked for is kept
    if (jfn && bpc == 0) {
        // the specialised sector kernels hold few enough registers for four
        // waves per SIMD; 16 workgroups per CU fill whole residency rounds
        bpc = 16;
    }
    return plan_launch(p, pk, fn, jfn, T, bpc, min_points);
}

qmc_status plan_collect(qmc_plan_s *p, uint32_t np, qmc_result *out, double *per_shift, bool crossing) {
    hipError_t e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) return hip_fail(e, "synchronize");
    if (p->timing) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, p->ev0, p->ev1) == hipSuccess) {
            p->kernel_ms += ms;
            p->kernel_launches += 1;
        }
    }
    return plan_results(p, np, out, per_shift, crossing);
}

// The result of an estimate whose output is in the plan's pinned mirror.
qmc_status plan_results(qmc_plan_s *p, uint32_t np, qmc_result *out, double *per_shift, bool crossing) {
    // with a crossing count the last of the np parts is the count, not a
    // value: it is left out of per_shift and of the finiteness check
    const uint32_t nv = crossing ? np - 1 : np;
    const double *q = p->h_out, *res = p->h_out + out_res_offset(p->m);
    bool finite = true;
    for (uint32_t k = 0; k < p->m; ++k)
        for (uint32_t j = 0; j < nv; ++j) {
            const double v = q[(size_t)k * np + j];
            finite = finite && std::isfinite(v);
            if (per_shift) per_shift[(size_t)k * nv + j] = v;
        }
    double crossed = 0.0;
    if (crossing) {
        // finalize scaled every part by the transform's constant and 1/n
        long double s = 0.0L;
        for (uint32_t k = 0; k < p->m; ++k) s += q[(size_t)k * np + nv];
        crossed = (double)(s / ((long double)p->m * transform_scale(p->tr, p->d)));
    }
    out->is_complex = nv >= 2;
    out->used_cv = 0;
    out->contour_crossed = crossed;
    if (!finite) {
        out->mean_re = out->mean_im = out->err_re = out->err_im = NAN;
        return fail(QMC_ENONFINITE, "a per-shift sum is not finite");
    }
    out->mean_re = res[0];
    out->mean_im = nv >= 2 ? res[1] : 0.0;
    out->err_re = res[2];
    out->err_im = nv >= 2 ? res[3] : 0.0;
    if (crossed > 0.0)
        return fail(QMC_ECONTOUR, "the deformed contour has Im(F - i delta) > 0 at a fraction %.3g of the points",
                    crossed);
    return QMC_OK;
}

// The conditions of a rule (eq. (2)) every entry point that takes one
// checks before any device call; t.alpha is cleared for transforms
// without a parameter.
qmc_status validate_rule(uint32_t d, uint64_t n, const uint64_t *g, uint32_t m, const double *shifts,
                         qmc_transform &t) {
    if (d == 0) return fail(QMC_EINVAL, "d must be >= 1");
    if (d > kMaxDim) return fail(QMC_EUNSUPPORTED, "d = %u > %u", d, kMaxDim);
    if (n < 2) return fail(QMC_EINVAL, "n must be >= 2");
    if (n > (1ull << 31)) return fail(QMC_EUNSUPPORTED, "n > 2^31");
    if (!g) return fail(QMC_EINVAL, "g is NULL");
    for (uint32_t i = 0; i < d; ++i)
        if (g[i] % n == 0) return fail(QMC_EINVAL, "g_%u mod n == 0", i);
    if (m < 2) return fail(QMC_EINVAL, "m must be >= 2 (eq. (3) divides by m - 1)");
    if (m > kMaxRows) return fail(QMC_EUNSUPPORTED, "m > %u", kMaxRows);
    if (!shifts) return fail(QMC_EINVAL, "shifts is NULL");
    for (size_t i = 0; i < (size_t)m * d; ++i)
        if (!(shifts[i] >= 0.0 && shifts[i] < 1.0)) return fail(QMC_EINVAL, "shift %zu outside [0,1)", i);
    if (t.kind != QMC_T_NONE && t.kind != QMC_T_KOROBOV && t.kind != QMC_T_BAKER && t.kind != QMC_T_SIDI)
        return fail(QMC_EINVAL, "unknown transform %d", t.kind);
    if (t.kind == QMC_T_KOROBOV && t.alpha < 1) return fail(QMC_EINVAL, "Korobov weight must be >= 1");
    if (t.kind == QMC_T_KOROBOV && t.alpha > 6) return fail(QMC_EUNSUPPORTED, "Korobov weight > 6");
    if (t.kind == QMC_T_SIDI && t.alpha < 1) return fail(QMC_EINVAL, "Sidi order must be >= 1");
    if (t.kind == QMC_T_SIDI && t.alpha > 6) return fail(QMC_EUNSUPPORTED, "Sidi order > 6");
    if (t.kind != QMC_T_KOROBOV && t.kind != QMC_T_SIDI) t.alpha = 0;
    return QMC_OK;
}

}  // namespace qmc

using namespace qmc;

// ==================================================================== C ABI
extern "C" {

const char *qmc_status_string(int32_t status) {
    // an int, not the enum: any value a caller passes is defined behaviour
    switch (status) {
    case QMC_OK: return "ok";
    case QMC_EINVAL: return "invalid argument";
    case QMC_EUNSUPPORTED: return "unsupported";
    case QMC_ENOMEM: return "out of memory";
    case QMC_EDEVICE: return "device error";
    case QMC_ENONFINITE: return "non-finite result";
    case QMC_ECONTOUR: return "deformed contour crosses the cut";
    }
    return "unknown status";
}

const char *qmc_last_error(void) { return g_last_error.c_str(); }

qmc_status qmc_plan_create(uint32_t d, uint64_t n, const uint64_t *g, uint32_t m, const double *shifts,
                           qmc_transform t, qmc_plan_t *out) {
    if (!out) return fail(QMC_EINVAL, "out is NULL");
    qmc_status vs = validate_rule(d, n, g, m, shifts, t);
    if (vs) return vs;

    auto *p = new (std::nothrow) qmc_plan_s();
    if (!p) return fail(QMC_ENOMEM, "host allocation");
    p->d = d;
    p->n = (uint32_t)n;
    p->m = m;
    p->inv_n = 1.0 / (double)n;
    p->tr = t;
    p->g.resize(d);
    for (uint32_t i = 0; i < d; ++i) p->g[i] = (uint32_t)(g[i] % n);
    p->shifts.assign(shifts, shifts + (size_t)m * d);
    hipError_t e = hipGetDevice(&p->device);
    if (e != hipSuccess) {
        delete p;
        return hip_fail(e, "hipGetDevice");
    }
    qmc_status st = QMC_OK;
    size_t cap = 0;
    if ((st = ensure_buffer((void **)&p->d_g, cap, d * sizeof(uint32_t), "g")) ||
        (cap = 0, st = ensure_buffer((void **)&p->d_gstep, cap, d * sizeof(uint32_t), "gstep")) ||
        (cap = 0, st = ensure_buffer((void **)&p->d_shifts, cap, (size_t)padded_rows(m) * d * sizeof(double),
                                     "shifts"))) {
        qmc_plan_destroy(p);
        return st;
    }
    e = hipHostMalloc((void **)&p->h_out, out_doubles(m) * sizeof(double), hipHostMallocDefault);
    if (e != hipSuccess) {
        qmc_plan_destroy(p);
        return fail(QMC_ENOMEM, "hipHostMalloc: %s", hipGetErrorString(e));
    }
    if ((e = hipMemcpy(p->d_g, p->g.data(), d * sizeof(uint32_t), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(p->d_shifts, padded_shifts(p->shifts, m, d, padded_rows(m), p->tr).data(),
                       (size_t)padded_rows(m) * d * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipEventCreate(&p->ev0)) != hipSuccess || (e = hipEventCreate(&p->ev1)) != hipSuccess) {
        qmc_plan_destroy(p);
        return hip_fail(e, "plan setup");
    }
    *out = p;
    return QMC_OK;
}

void qmc_plan_destroy(qmc_plan_t p) {
    if (!p) return;
    if (p->stream) hipStreamSynchronize(p->stream);
    else hipDeviceSynchronize();
    plan_release_extra(p);
    if (p->d_g) hipFree(p->d_g);
    if (p->d_gstep) hipFree(p->d_gstep);
    if (p->d_shifts) hipFree(p->d_shifts);
    if (p->d_params) hipFree(p->d_params);
    if (p->d_partials) hipFree(p->d_partials);
    if (p->h_out) hipHostFree(p->h_out);
    if (p->ev0) hipEventDestroy(p->ev0);
    if (p->ev1) hipEventDestroy(p->ev1);
    delete p;
}

qmc_status qmc_plan_set_stream(qmc_plan_t p, void *stream) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    p->stream = (hipStream_t)stream;
    return QMC_OK;
}

qmc_status qmc_plan_set_launch(qmc_plan_t p, const qmc_launch *cfg) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (!cfg) {
        p->launch = qmc_launch{0, 0};
        return QMC_OK;
    }
    const uint32_t T = cfg->shift_tile;
    if (T != 0 && T != 1 && T != 2 && T != 4 && T != 8) return fail(QMC_EINVAL, "shift_tile must be 1, 2, 4 or 8");
    if (cfg->blocks_per_cu > 1024) return fail(QMC_EINVAL, "blocks_per_cu > 1024");
    p->launch = *cfg;
    return QMC_OK;
}

qmc_status qmc_plan_set_jit(qmc_plan_t p, int32_t mode) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (mode < 0 || mode > 2) return fail(QMC_EINVAL, "jit mode must be 0, 1 or 2");
    p->jit_mode = mode;
    return QMC_OK;
}

qmc_status qmc_plan_get_launch(qmc_plan_t p, qmc_launch *cfg, int32_t *used_jit) {
    if (!p || !cfg) return fail(QMC_EINVAL, "null argument");
    cfg->shift_tile = p->last_T;
    cfg->blocks_per_cu = p->last_bx;
    if (used_jit) *used_jit = p->last_jit ? 1 : 0;
    return QMC_OK;
}

qmc_status qmc_plan_set_timing(qmc_plan_t p, int32_t enable) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    p->timing = enable != 0;
    return QMC_OK;
}

qmc_status qmc_plan_kernel_time(qmc_plan_t p, double *total_ms, uint64_t *launches, int32_t reset) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (total_ms) *total_ms = p->kernel_ms;
    if (launches) *launches = p->kernel_launches;
    if (reset) {
        p->kernel_ms = 0.0;
        p->kernel_launches = 0;
    }
    return QMC_OK;
}

qmc_status qmc_integrate(qmc_plan_t p, qmc_family family, const void *params, qmc_result *out,
                         double *per_shift) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (!out) return fail(QMC_EINVAL, "out is NULL");
    const Packed *ppk;
    qmc_status st = plan_pack(p, (int)family, params, ppk);
    if (st) return st;
    const Packed &pk = *ppk;
    if (pk.orders >= 2) return fail(QMC_EINVAL, "n_orders >= 2: use qmc_integrate_orders");
    qmc_launch L = p->launch;
    if (L.shift_tile == 0 && L.blocks_per_cu == 0) {
        const bool sector = pk.key_family == QMC_F_SECTOR || pk.key_family == kFamSectorComplex;
        qmc_launch tuned;
        if (tune_lookup(p, pk, sector && p->jit_mode != 0, tuned)) L = tuned;
    }
    if ((st = plan_enqueue(p, pk, L.shift_tile, L.blocks_per_cu))) return st;
    return plan_collect(p, pk.np, out, per_shift, pk.crossing);
}

qmc_status qmc_integrate_orders(qmc_plan_t p, qmc_family family, const void *params, qmc_result *out,
                                double *per_shift) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (!out) return fail(QMC_EINVAL, "out is NULL");
    if (family != QMC_F_SECTOR) return fail(QMC_EUNSUPPORTED, "expansion orders are built for QMC_F_SECTOR");
    const Packed *ppk;
    qmc_status st = plan_pack(p, (int)family, params, ppk);
    if (st) return st;
    const Packed &pk = *ppk;
    const uint32_t no = pk.orders >= 2 ? pk.orders : 1u;
    if ((st = plan_enqueue(p, pk, p->launch.shift_tile, p->launch.blocks_per_cu))) return st;
    qmc_result first;
    st = plan_collect(p, pk.np, &first, per_shift, pk.crossing);
    if (st && st != QMC_ENONFINITE && st != QMC_ECONTOUR) return st;
    const double *res = p->h_out + out_res_offset(p->m);
    for (uint32_t k = 0; k < no; ++k) {
        if (pk.cplx) {  // parts (2k, 2k+1) = (Re, Im) of order k form pair k
            out[k] = qmc_result{res[4 * k], res[4 * k + 1], res[4 * k + 2], res[4 * k + 3], 1, 0, 0.0};
        } else {        // part k = order k, pairs of orders share a result block
            const uint32_t b = 4 * (k / 2), o = k % 2;
            out[k] = qmc_result{res[b + o], 0.0, res[b + 2 + o], 0.0, 0, 0, 0.0};
        }
        if (st == QMC_ENONFINITE) out[k] = qmc_result{NAN, NAN, NAN, NAN, pk.cplx ? 1 : 0, 0, 0.0};
        out[k].contour_crossed = first.contour_crossed;
    }
    return st;
}

qmc_status qmc_integrate_sum(qmc_plan_t p, uint32_t count, const qmc_sector_params *const *params, qmc_result *out,
                             double *per_shift) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (!params || !out) return fail(QMC_EINVAL, "null argument");
    if (count == 0) return fail(QMC_EINVAL, "count must be >= 1");
    if (count > kMaxSumSectors) return fail(QMC_EUNSUPPORTED, "more than %u sectors in one sum", kMaxSumSectors);
    Packed sum;
    std::vector<size_t> offs;
    for (uint32_t i = 0; i < count; ++i) {
        if (!params[i]) return fail(QMC_EINVAL, "params[%u] is NULL", i);
        Packed pk;
        qmc_status st = pack_params(QMC_F_SECTOR, p->d, params[i], pk);
        if (st) return st;
        if (pk.orders >= 2 || pk.deform)
            return fail(QMC_EUNSUPPORTED, "sums take plain sectors (n_orders < 2, deform_lambda = 0)");
        if (i == 0) {
            sum.np = pk.np;
            sum.cplx = pk.cplx;
            sum.key_family = pk.key_family;
        } else if (pk.cplx != sum.cplx) {
            return fail(QMC_EINVAL, "mixed real and complex sectors");
        }
        offs.push_back(sum.blob.size());
        sum.blob.insert(sum.blob.end(), pk.blob.begin(), pk.blob.end());
    }
    const uint32_t T = p->launch.shift_tile ? p->launch.shift_tile : 2u;
    std::string err;
    hipFunction_t jfn = jit_sum_kernel(sum.blob, offs, p->d, p->tr, T, sum.cplx, p->device, err);
    if (!jfn) return fail(QMC_EUNSUPPORTED, "specialised sum kernel: %s", err.c_str());
    const uint32_t bpc = p->launch.blocks_per_cu;
    qmc_status st = plan_launch(p, sum, nullptr, jfn, T, bpc ? bpc : 16, bpc ? 4 : 32);
    if (st) return st;
    return plan_collect(p, sum.np, out, per_shift);
}

qmc_status qmc_deform_check(qmc_plan_t p, const qmc_sector_params *params, double *fraction, double *per_shift) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (!fraction || !params) return fail(QMC_EINVAL, "null argument");
    if (params->deform_lambda == 0.0) return fail(QMC_EINVAL, "deform_lambda is 0");
    Packed pk;
    qmc_status st = pack_params(QMC_F_SECTOR, p->d, params, pk);
    if (st) return st;
    // the check functor: one real part, 1 where Im(F(z) - i delta) > 0
    uint64_t flags;
    std::memcpy(&flags, &pk.blob[2], sizeof flags);
    pk.blob[2] = bits(flags | kSectorDeformCheck);
    pk.np = 1;
    pk.cplx = false;
    pk.crossing = false;
    pk.orders = 0;
    if ((st = plan_enqueue(p, pk, p->launch.shift_tile, p->launch.blocks_per_cu))) return st;
    qmc_result r;
    st = plan_collect(p, 1, &r, per_shift);
    if (st) return st;
    // finalize multiplies every sum by the transform's constant
    const double scale = transform_scale(p->tr, p->d);
    *fraction = r.mean_re / scale;
    if (per_shift)
        for (uint32_t k = 0; k < p->m; ++k) per_shift[k] /= scale;
    return QMC_OK;
}

qmc_status qmc_deform_select(qmc_plan_t p, const qmc_sector_params *params, double lam_max, double shrink,
                             uint32_t count, double *lam_out, qmc_result *out) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (!params || !lam_out || !out) return fail(QMC_EINVAL, "null argument");
    if (!(lam_max > 0.0) || !std::isfinite(lam_max)) return fail(QMC_EINVAL, "lam_max must be positive and finite");
    if (!(shrink > 0.0 && shrink < 1.0)) return fail(QMC_EINVAL, "shrink must lie in (0, 1)");
    if (count == 0 || count > 64) return fail(QMC_EINVAL, "count must be 1..64");
    if (params->n_orders >= 2) return fail(QMC_EINVAL, "select lambda on the plain integrand (n_orders < 2)");
    qmc_sector_params q = *params;
    bool found = false;
    double best_err = 0.0;
    double lam = lam_max;
    for (uint32_t i = 0; i < count; ++i, lam *= shrink) {
        q.deform_lambda = lam;
        double frac;
        qmc_status st = qmc_deform_check(p, &q, &frac, nullptr);
        if (st) return st;
        if (frac > 0.0) continue;
        qmc_result r;
        st = qmc_integrate(p, QMC_F_SECTOR, &q, &r, nullptr);
        if (st == QMC_ENONFINITE || st == QMC_ECONTOUR) continue;
        if (st) return st;
        const double err = std::hypot(r.err_re, r.err_im);
        if (!found || err < best_err) {
            found = true;
            best_err = err;
            *lam_out = lam;
            *out = r;
        }
    }
    if (!found) return fail(QMC_EUNSUPPORTED, "every lambda of the ladder crosses the -i0 side or is not finite");
    return QMC_OK;
}

qmc_status qmc_math_eval(int32_t fn, uint64_t count, const double *x, double *y) {
    if (fn < 0 || fn > 6)
        return fail(QMC_EINVAL, "fn must be 0 (log), 1 (exp), 2 (atan2), 3 (sincos), 4 (log512), 5 (exp512) or 6 (phase)");
    if (count && (!x || !y)) return fail(QMC_EINVAL, "null array");
    if (count > (1ull << 28)) return fail(QMC_EINVAL, "count > 2^28");
    if (count == 0) return QMC_OK;
    const size_t nx = fn == 2 ? 2 * count : count, ny = fn == 3 || fn == 6 ? 2 * count : count;
    DeviceScratch s;
    qmc_status st;
    if ((st = s.alloc(nx * 8)) || (st = s.alloc(ny * 8))) return st;
    hipError_t e = hipMemcpy(s.ptr[0], x, nx * 8, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = launch_math(fn, count, (const double *)s.ptr[0], (double *)s.ptr[1], nullptr);
    if (e == hipSuccess) e = hipMemcpy(y, s.ptr[1], ny * 8, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "math eval");
    return QMC_OK;
}

qmc_status qmc_korobov_vector(uint64_t n, uint32_t d, uint64_t a, uint64_t *g) {
    if (!g) return fail(QMC_EINVAL, "g is NULL");
    if (n < 2 || d == 0) return fail(QMC_EINVAL, "need n >= 2 and d >= 1");
    if (n > (1ull << 32)) return fail(QMC_EUNSUPPORTED, "n > 2^32");
    uint64_t v = 1 % n;
    a %= n;
    for (uint32_t i = 0; i < d; ++i) {
        g[i] = v;
        v = (v * a) % n;
    }
    return QMC_OK;
}

qmc_status qmc_lattice_dump(qmc_plan_t p, uint64_t j_lo, uint64_t count, uint32_t *idx_out, uint64_t *sums_out) {
    if (!p) return fail(QMC_EINVAL, "plan is NULL");
    if (count && !idx_out) return fail(QMC_EINVAL, "idx_out is NULL");
    if (count > (1ull << 24)) return fail(QMC_EINVAL, "count > 2^24");
    if (j_lo + count > p->n) return fail(QMC_EINVAL, "j range beyond n");
    // same grid as the lattice kernel's default launch for a real family
    const uint32_t T = p->launch.shift_tile ? p->launch.shift_tile : 1;
    const uint32_t tiles = (p->m + T - 1) / T;
    const uint32_t bx = grid_x(p->n, tiles, p->device, p->launch.blocks_per_cu);
    qmc_status st = plan_set_gstep(p, bx * kBlock);
    if (st) return st;
    uint32_t *d_idx = nullptr;
    unsigned long long *d_sums = nullptr;
    hipError_t e;
    if ((e = hipMalloc(&d_sums, 2 * p->d * sizeof(unsigned long long))) != hipSuccess)
        return fail(QMC_ENOMEM, "hipMalloc sums");
    if (count && (e = hipMalloc(&d_idx, count * p->d * sizeof(uint32_t))) != hipSuccess) {
        hipFree(d_sums);
        return fail(QMC_ENOMEM, "hipMalloc idx");
    }
    e = hipMemsetAsync(d_sums, 0, 2 * p->d * sizeof(unsigned long long), p->stream);
    DumpArgs a{};
    a.n = p->n;
    a.d = p->d;
    a.inv_n = p->inv_n;
    a.g = p->d_g;
    a.gstep = p->d_gstep;
    a.j_lo = j_lo;
    a.j_hi = j_lo + count;
    a.idx_out = d_idx;
    a.sums = d_sums;
    if (e == hipSuccess) e = launch_dump(a, bx, p->stream);
    if (e == hipSuccess && count)
        e = hipMemcpyAsync(idx_out, d_idx, count * p->d * sizeof(uint32_t), hipMemcpyDeviceToHost, p->stream);
    std::vector<unsigned long long> sums(2 * p->d);
    if (e == hipSuccess)
        e = hipMemcpyAsync(sums.data(), d_sums, 2 * p->d * sizeof(unsigned long long), hipMemcpyDeviceToHost,
                           p->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
    hipFree(d_sums);
    if (d_idx) hipFree(d_idx);
    if (e != hipSuccess) return hip_fail(e, "lattice dump");
    if (sums_out)
        for (uint32_t i = 0; i < 2 * p->d; ++i) sums_out[i] = sums[i];
    return QMC_OK;
}

}  // extern "C"
