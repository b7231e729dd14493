// Device helpers shared by the Vecchia kernels: covariance closed forms,
// parameter unpacking, deterministic wave/block reductions and compensated
// (double-double) accumulation.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "exp_table.h"
#include "log_table.h"

namespace vecchia {

constexpr int kWave = 64;                     // CDNA wavefront width
constexpr double kLog2Pi = 1.8378770664093454835606594728112;
constexpr int64_t kNoFailure = INT64_MAX;     // "no failing point" sentinel in partial status words
constexpr int kChunk = 16;                    // conditionals summed per partial (fixed: fixes the summation order)

// Covariance parameters as the kernels use them; alpha is the exponent of
// the power exponential (unused by the Matern codes).
struct Params {
    double sigma2, beta, tau2, inv_beta, alpha;
    bool valid;
};

__device__ inline Params load_params(const double *__restrict__ theta, double alpha = 1.0) {
    Params p;
    p.sigma2 = theta[0];
    p.beta = theta[1];
    p.tau2 = theta[2];
    p.valid = (p.sigma2 > 0.0) && (p.beta > 0.0) && (p.tau2 >= 0.0) && isfinite(p.sigma2) && isfinite(p.beta) &&
              isfinite(p.tau2);
    p.inv_beta = 1.0 / p.beta;
    p.alpha = alpha;
    return p;
}

// Covariance codes of the kernels: KC = family + 4 * metric, family 0, 1, 2
// for Matern nu = 1/2, 3/2, 5/2 (Eq. (2)) and 3 for the power exponential
// sigma2 exp(-d^alpha / beta) (Sec. V-C); metric 0 Euclidean on (x, y), 1
// great-circle on (longitude, latitude) in degrees, in kilometres.
__host__ __device__ constexpr int kc_family(int KC) { return KC & 3; }
__host__ __device__ constexpr bool kc_gcd(int KC) { return (KC >> 2) != 0; }
constexpr double kEarthRadiusKm = 6371.0;
constexpr double kDeg2Rad = 0.017453292519943295769236907684886;

// e^{-r} for r >= 0.  Range reduction x = -r = k ln2 + f with |f| <= ln2/2
// (ln2 split into a head with trailing zero bits and a tail, so k*ln2_head is
// exact), e^f by its Taylor polynomial of degree 13 (truncation below 6e-18
// relative), then scaling by 2^k.  Results below the double range flush to
// 0; NaN propagates.  About 19 instructions, no table.
__device__ __forceinline__ double exp_neg(double r) {
    double x = -r;
    x = (x < -745.5) ? -745.5 : x;  // keeps NaN (the comparison is false)
    const double k = __builtin_rint(x * 1.4426950408889634074);
    double f = fma(k, -6.93147180369123816490e-01, x);
    f = fma(k, -1.90821492927058770002e-10, f);
    double p = 1.0 / 6227020800.0;          // 1/13!
    p = fma(p, f, 1.0 / 479001600.0);       // 1/12!
    p = fma(p, f, 1.0 / 39916800.0);        // 1/11!
    p = fma(p, f, 1.0 / 3628800.0);         // 1/10!
    p = fma(p, f, 1.0 / 362880.0);          // 1/9!
    p = fma(p, f, 1.0 / 40320.0);           // 1/8!
    p = fma(p, f, 1.0 / 5040.0);            // 1/7!
    p = fma(p, f, 1.0 / 720.0);             // 1/6!
    p = fma(p, f, 1.0 / 120.0);             // 1/5!
    p = fma(p, f, 1.0 / 24.0);              // 1/4!
    p = fma(p, f, 1.0 / 6.0);               // 1/3!
    p = fma(p, f, 0.5);
    p = fma(p, f, 1.0);
    p = fma(p, f, 1.0);
    return __builtin_ldexp(p, (int)k);
}

// sqrt(s) for a squared distance s >= 0: hardware reciprocal square root and
// two coupled Newton (Goldschmidt) refinements of sqrt and 1/(2 sqrt), as in
// a correctly rounded software sqrt, without the denormal rescaling: s below
// 1e-290 (coincident points up to 1e-145) gives 0.  NaN propagates.
__device__ __forceinline__ double sqrt_dist(double s) {
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y;
    double h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    const double d = fma(-g, g, s);
    g = fma(d, h, g);
    return (s > 1e-290) ? g : ((s >= 0.0) ? 0.0 : s);
}

// e^{-r} for r >= 0 by Tang's table-driven method: -r = (64 k + j) ln2/64 + f
// with |f| <= ln2/128, so e^{-r} = 2^k 2^{j/64} e^f.  `tab` holds 2^{j/64}
// as hi + lo pairs (kExp2Frac64, staged in LDS by the caller); q = e^f - 1 by
// its Taylor polynomial of degree 6 (truncation below 3e-20), and the result
// hi + (lo + hi q) rounds once at the end, so the error stays just above half
// an ulp.  ln2/64 is split into a 36-bit head (n ln2/64 exact for |n| < 2^17)
// and a tail.  Arguments beyond 746 give 0; a NaN argument gives 0 as well,
// so callers validate their inputs instead.
__device__ __forceinline__ double exp_neg_tab(double r, const double *tab) {
    const double x = fmax(-r, -746.0);
    const double nf = __builtin_rint(x * 0x1.71547652b82fep+6);  // 64 / ln2
    const int n = (int)nf;
    double f = fma(nf, -0x1.62e42fefa0000p-7, x);  // head of ln2/64
    f = fma(nf, -0x1.cf79abc9e3b3ap-46, f);        // tail of ln2/64
    double q = fma(f, 1.0 / 720.0, 1.0 / 120.0);
    q = fma(q, f, 1.0 / 24.0);
    q = fma(q, f, 1.0 / 6.0);
    q = fma(q, f, 0.5);
    q = fma(q, f, 1.0);
    q *= f;  // e^f - 1
    const double2 t = *reinterpret_cast<const double2 *>(tab + 2 * (n & 63));
    return __builtin_ldexp(t.x + fma(t.x, q, t.y), n >> 6);
}

// sin x.  Neighbouring points give half-angle differences far below 0.25
// rad, where the Taylor polynomial to x^13 is used (truncation below 1e-21
// relative, Horner in x^2, one rounding at the end); larger arguments take
// the library sine.
__device__ __forceinline__ double sin_short(double x) {
    if (fabs(x) <= 0.25) {
        const double x2 = x * x;
        double q = 1.0 / 6227020800.0;   // 1/13!
        q = fma(q, x2, -1.0 / 39916800.0);  // -1/11!
        q = fma(q, x2, 1.0 / 362880.0);     // 1/9!
        q = fma(q, x2, -1.0 / 5040.0);      // -1/7!
        q = fma(q, x2, 1.0 / 120.0);        // 1/5!
        q = fma(q, x2, -1.0 / 6.0);         // -1/3!
        return fma(x * x2, q, x);
    }
    return sin(x);
}

// asin(sqrt(h)) for 0 <= h <= 1.  For h <= 0.01 (great-circle distances up
// to about 1270 km) the series asin s = s (1 + sum_n c_n s^2n), c_n =
// (2n)! / (4^n (n!)^2 (2n + 1)), to n = 8 (truncation below 2e-18
// relative); otherwise the library asin.
__device__ __forceinline__ double asin_sqrt(double h) {
    const double s = sqrt(h);
    if (h <= 0.01) {
        double p = 6435.0 / 557056.0;
        p = fma(p, h, 143.0 / 10240.0);
        p = fma(p, h, 231.0 / 13312.0);
        p = fma(p, h, 63.0 / 2816.0);
        p = fma(p, h, 35.0 / 1152.0);
        p = fma(p, h, 5.0 / 112.0);
        p = fma(p, h, 3.0 / 40.0);
        p = fma(p, h, 1.0 / 6.0);
        return fma(s * h, p, s);
    }
    return asin(s);
}

// Great-circle distance in km between (lon, lat) points a and b in degrees,
// given cos(lat) of each: hav(d / R) = hav(dlat) + cos lat_a cos lat_b hav(dlon)
// with hav(t) = sin^2(t / 2), differences taken in degrees first.  Coincident
// points give exactly 0.
__device__ __forceinline__ double gcd_km(double lona, double lata, double ca, double lonb, double latb, double cb) {
    const double s1 = sin_short(0.5 * ((lata - latb) * kDeg2Rad));
    const double s2 = sin_short(0.5 * ((lona - lonb) * kDeg2Rad));
    const double h = fmin(fma(s1, s1, (ca * cb) * (s2 * s2)), 1.0);
    return (2.0 * kEarthRadiusKm) * asin_sqrt(h);
}

// The parameter-free part of the scaled distance: d (Matern) or d^alpha
// (power exponential; alpha = 1 and 2 without the exponential, otherwise
// e^(alpha ln d) with the table exponential, and 0 for d = 0).  alpha is
// fixed per call, so this is shared by every (sigma2, beta, tau2).
template <int KC>
__device__ __forceinline__ double dist_pow(double d, const Params &P, const double *tab) {
    if constexpr (kc_family(KC) == 3) {
        double da;
        if (P.alpha == 1.0) {
            da = d;
        } else if (P.alpha == 2.0) {
            da = d * d;
        } else {
            da = (d > 0.0) ? exp_neg_tab(-(P.alpha * log(d)), tab) : 0.0;
        }
        return da;
    } else {
        return d;
    }
}

// Scaled distance r fed to the closed forms: d / beta (Matern) or
// d^alpha / beta (power exponential).
template <int KC>
__device__ __forceinline__ double cov_scaled(double d, const Params &P, const double *tab) {
    return dist_pow<KC>(d, P, tab) * P.inv_beta;
}

// ---- the tiled kernel's forms -------------------------------------------------
//
// The exponential of exp_neg_tab rearranged for fewer instructions (17 against
// 22 with the table's address; the tiled kernels evaluate it for every pair
// and are bound by vector issue).  Entry j of the staged table holds hi =
// 2^(j/64) and lo / hi, so that the low part joins e^f - 1 in the polynomial's
// last step.  n = rint(64 x / ln2) is the low word of 64 x / ln2 + 1.5 2^52.
__device__ __forceinline__ void stage_exp_entry(int j, double *tab) {
    const ExpTableEntry e = kExp2Frac64[j];
    tab[2 * j] = e.hi;
    tab[2 * j + 1] = e.lo * __builtin_amdgcn_rcp(e.hi);  // |lo / hi| < 2^-53: the estimate is plenty
}

// Constants of the covariance evaluation.  A vector instruction reads at most
// one constant from scalar registers, and a constant in a vector register is
// otherwise built again (two moves) in every basic block: PIN keeps the three
// that meet another constant, or are overwritten by a fused multiply-add, in
// vector registers of their own, and the rest in scalar registers.
struct CovConst {
    double eps, magic, c120;                                      // vector
    double unmagic, inv_ln2_64, head, tail, c720, c24, c6, rmax;  // scalar
};
template <bool PIN>
__device__ __forceinline__ CovConst cov_const() {
    CovConst c{0x1p-1000, 0x1.8p52, 1.0 / 120.0, -0x1.8p52, -0x1.71547652b82fep+6, -0x1.62e42fefa0000p-7,
               -0x1.cf79abc9e3b3ap-46, 1.0 / 720.0, 1.0 / 24.0, 1.0 / 6.0, 746.0};
    if constexpr (PIN) {
        asm volatile("" : "+v"(c.eps), "+v"(c.magic), "+v"(c.c120));
        asm volatile("" : "+s"(c.unmagic), "+s"(c.inv_ln2_64), "+s"(c.head), "+s"(c.tail));
        asm volatile("" : "+s"(c.c720), "+s"(c.c24), "+s"(c.c6), "+s"(c.rmax));
    }
    return c;
}

// A staged table by its LDS address in a scalar register, opaque to the
// compiler: it would otherwise add the (zero) base of the dynamic LDS to every
// entry's address in an instruction of its own.
typedef const __attribute__((address_space(3))) double *LdsTab;
typedef double dvec2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ LdsTab lds_table(const double *tab) {
    uint32_t a = (uint32_t)(uintptr_t)(LdsTab)tab;
    asm volatile("" : "+s"(a));
    return (LdsTab)(uintptr_t)a;
}
// entry j (two doubles)
__device__ __forceinline__ dvec2 table_entry(LdsTab tab, uint32_t j) {
    uint32_t a;
    asm("v_lshl_add_u32 %0, %1, 4, %2" : "=v"(a) : "v"(j), "s"((uint32_t)(uintptr_t)tab));
    return *(const __attribute__((address_space(3))) dvec2 *)(uintptr_t)a;
}

// e^-r for -709 <= r <= 746, one rounding at the end (just above half an ulp,
// as exp_neg_tab) and another below the normal range; 0 at 746, where
// scaled_dist stops.  e^f - 1 is exp_neg_tab's Taylor polynomial: one of degree
// 5 with Chebyshev coefficients is an instruction less, but 0.514 ulp at worst
// where this is 0.504.
__device__ __forceinline__ double exp_neg_staged(double r, LdsTab tab, const CovConst &c) {
    const double t = fma(r, c.inv_ln2_64, c.magic);
    const int n = __double2loint(t);
    const double nf = t + c.unmagic;
    double f = fma(nf, c.head, -r);
    f = fma(nf, c.tail, f);
    double q = fma(f, c.c720, c.c120);
    q = fma(q, f, c.c24);
    q = fma(q, f, c.c6);
    q = fma(q, f, 0.5);
    q = fma(q, f, 1.0);
    const dvec2 e = table_entry(tab, n & 63);
    return __builtin_ldexp(fma(e.x, fma(q, f, e.y), e.x), n >> 6);
}

// Distance of two points from their coordinate differences, without a branch:
// the square is raised by 2^-1000 (below half an ulp of any square from 2^-946
// up, so other distances are unchanged) so that the reciprocal square root
// never sees 0; coincident points get distance 2^-500, whose covariance is the
// zero-distance value to the last bit.  One coupled Newton step and one
// correction by the residual, as in sqrt_dist, but without the refinement of
// 1/(2 sqrt): the correction is a factor 2^-47 of the result and the hardware
// estimate serves it.
__device__ __forceinline__ double dist_pos(double dx, double dy, const CovConst &c) {
    const double s = fma(dx, dx, fma(dy, dy, c.eps));
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y;
    const double h = 0.5 * y;
    g = fma(g, fma(-h, g, 0.5), g);
    return fma(fma(-g, g, s), h, g);
}

// log x for positive normal x: x = 2^e m with m in [sqrt(1/2), sqrt 2),
// log m = 2 atanh(s), s = (m - 1) / (m + 1), by the odd Taylor series to s^21
// (truncation below 2^-55 relative at |s| <= 0.1716).  About 40 instructions;
// NaN and non-positive arguments give NaN.
__device__ __forceinline__ double log_pos(double x) {
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0x1.6a09e667f3bcdp-1;
    m = low ? m + m : m;
    e = low ? e - 1 : e;
    const double f = m - 1.0, d = m + 1.0;
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    y = fma(fma(-d, y, 1.0), y, y);
    double s = f * y;
    s = fma(fma(-s, d, f), y, s);
    const double z = s * s;
    double p = fma(z, 1.0 / 21.0, 1.0 / 19.0);
    p = fma(p, z, 1.0 / 17.0);
    p = fma(p, z, 1.0 / 15.0);
    p = fma(p, z, 1.0 / 13.0);
    p = fma(p, z, 1.0 / 11.0);
    p = fma(p, z, 1.0 / 9.0);
    p = fma(p, z, 1.0 / 7.0);
    p = fma(p, z, 1.0 / 5.0);
    p = fma(p, z, 1.0 / 3.0);
    const double s2 = s + s;
    const double lm = fma(s2 * z, p, s2);
    const double k = (double)e;
    // ln2 as a 32-bit head (k head is exact) and a tail
    const double r = fma(k, 0x1.62e42fee00000p-1, fma(k, 0x1.a39ef35793c76p-33, lm));
    return x > 0.0 ? r : __builtin_nan("");
}

// Staged tables of the tiled and rows kernels: 64 entries of the exponential
// and, for the power exponential, 64 of the logarithm after them.
__host__ __device__ constexpr int staged_doubles(bool powexp) {
    return 2 * kExpTableSize + (powexp ? 2 * kLogTableSize : 0);
}
template <int KC>
__device__ __forceinline__ void stage_tables(int t, double *tab) {
    if (t < kExpTableSize) stage_exp_entry(t, tab);
    if constexpr (kc_family(KC) == 3) {
        if (t < kLogTableSize) {
            tab[2 * kExpTableSize + 2 * t] = kLogMant64[t].c;
            tab[2 * kExpTableSize + 2 * t + 1] = t < kLogLowEntries ? kLogMantLow[t] : kLogMant64[t].neg_log_c;
        }
    }
}

// log x + a b for positive normal x, to about half an ulp of the result plus
// 2^-54 (|a b| < 0.004; log x alone with a = 0), and within 2^-58 near 1, where the result is small (it feeds an
// exponential): x = 2^e m with m in [1/2, 1), r = m c - 1 with c near 1 / m
// (|r| <= 2^-7), log x = e ln2 - log c + log1p r, the last by its Taylor
// polynomial of degree 7 (truncation 2e-18).  Mantissas of the table's first
// entries count as 2 m and 2^(e - 1), so that no ln2 cancels near 1.
__device__ __forceinline__ double log_staged(double x, double a, double b, LdsTab tab) {
    const double m = __builtin_amdgcn_frexp_mant(x);
    const int hi = __double2hiint(x);
    const double k = (double)((hi - ((1022 << 20) + (kLogLowEntries << 14))) >> 20);
    const int j = (hi >> 14) & 63;
    const dvec2 e = table_entry(tab + 2 * kExpTableSize, j);
    const double r = fma(m, e.x, -1.0);
    double p = fma(r, 1.0 / 7.0, -1.0 / 6.0);
    p = fma(p, r, 1.0 / 5.0);
    p = fma(p, r, -1.0 / 4.0);
    p = fma(p, r, 1.0 / 3.0);
    p = fma(p, r, -0.5);
    p = fma(r * r, p, fma(a, b, r));
    // ln2 as a 32-bit head (k head is exact) and a tail
    return fma(k, 0x1.62e42fee00000p-1, e.y + fma(k, 0x1.a39ef35793c76p-33, p));
}

// sin x for |x| <= pi / 4 by its Taylor polynomial (truncation below 4e-17).
__device__ __forceinline__ double sin_quarter(double x) {
    const double z = x * x;
    double q = 1.0 / 355687428096000.0;  // 1/17!
    q = fma(q, z, -1.0 / 1307674368000.0);
    q = fma(q, z, 1.0 / 6227020800.0);
    q = fma(q, z, -1.0 / 39916800.0);
    q = fma(q, z, 1.0 / 362880.0);
    q = fma(q, z, -1.0 / 5040.0);
    q = fma(q, z, 1.0 / 120.0);
    q = fma(q, z, -1.0 / 6.0);
    return fma(x * z, q, x);
}

// |sin| and cos of an angle in degrees, any finite one: reduced in degrees,
// where every step is exact, to [0, 45] or its complement, sin(90 - b) = cos b
// = 1 - 2 sin^2(b / 2).  Little code and no stack frame, unlike the library's
// reduction, since it is inlined wherever a covariance is evaluated.
__device__ __forceinline__ double reduce_degrees(double a) {  // |a| folded into [0, 180]
    a = fabs(a);
    while (a > 180.0) a = fabs(fma(__builtin_rint(a * (1.0 / 360.0)), -360.0, a));
    return a;
}
__device__ __forceinline__ double sin_deg_90(double a) {  // a in [0, 90]
    const bool top = a > 45.0;
    const double s = sin_quarter((top ? 45.0 - 0.5 * a : a) * kDeg2Rad);
    return top ? fma(-2.0 * s, s, 1.0) : s;
}
__device__ __forceinline__ double abs_sin_deg(double a) {
    a = reduce_degrees(a);
    return sin_deg_90(a > 90.0 ? 180.0 - a : a);
}
__device__ __forceinline__ double cos_deg(double a) {
    a = reduce_degrees(a);
    const double c = sin_deg_90(fabs(90.0 - a));
    return a > 90.0 ? -c : c;
}

// sin x for |x| <= 0.25: sin_short's polynomial
__device__ __forceinline__ double sin_near(double x) {
    const double z = x * x;
    double q = 1.0 / 6227020800.0;  // 1/13!
    q = fma(q, z, -1.0 / 39916800.0);
    q = fma(q, z, 1.0 / 362880.0);
    q = fma(q, z, -1.0 / 5040.0);
    q = fma(q, z, 1.0 / 120.0);
    q = fma(q, z, -1.0 / 6.0);
    return fma(x * z, q, x);
}

// sqrt x for normal x, as dist_pos
__device__ __forceinline__ double sqrt_lean(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    const double h = 0.5 * y;
    g = fma(g, fma(-h, g, 0.5), g);
    return fma(fma(-g, g, x), h, g);
}

// The parameter-free part of the scaled distance for a pair of points (cos of
// the latitudes in ca, cb for the great-circle codes): d, or d^alpha for the
// power exponential (0 for coincident points: the power of the 2^-500 that
// stands for their distance need not be small).  The coordinates must be finite.
//
// Great-circle distances: h = hav(d / R) as in gcd_km, d = 2 R asin sqrt h by
// the series of asin(s) / s in h up to h = 0.01 (1270 km).  For the power exponential the
// square root is not taken: 2 ln d = ln(4 R^2 h) + 2 ln(asin(s) / s), the last
// by its own series in h (to h^7, truncation 8e-19), added before the
// logarithm's last rounding.
template <int KC>
__device__ __forceinline__ double pair_dist_pow(double xa, double ya, double ca, double xb, double yb, double cb,
                                                const Params &P, LdsTab tab, const CovConst &cc) {
    if constexpr (kc_gcd(KC)) {
        const double dy = ya - yb, dx = xa - xb;
        const double x1 = dy * (0.5 * kDeg2Rad), x2 = dx * (0.5 * kDeg2Rad);
        double s1 = sin_near(x1), s2 = sin_near(x2);
        if (fmax(fabs(x1), fabs(x2)) > 0.25) {
            s1 = abs_sin_deg(0.5 * dy);
            s2 = abs_sin_deg(0.5 * dx);
        }
        double h = fmin(fma(s1, s1, fma(ca * cb, s2 * s2, cc.eps)), 1.0);
        // far pairs: the angle is halved (h becomes h / (2 (1 + sqrt(1 - h))))
        // until the series holds
        double r2 = 2.0 * kEarthRadiusKm;
        if (h > 0.01) {
            do {
                const double u = 1.0 + sqrt_lean(fma(-1.0, h, 1.0) + 0x1p-1000);
                h = (0.5 * h) / u;
                r2 += r2;
            } while (h > 0.01);
        }
        if constexpr (kc_family(KC) == 3) {
            if (P.alpha != 1.0 && P.alpha != 2.0) {
                double p = 36740617.0 / 3831077250.0;
                p = fma(p, h, 92427157.0 / 7662154500.0);
                p = fma(p, h, 14797.0 / 935550.0);
                p = fma(p, h, 2497.0 / 113400.0);
                p = fma(p, h, 191.0 / 5670.0);
                p = fma(p, h, 11.0 / 180.0);
                p = fma(p, h, 1.0 / 6.0);
                const double lnd2 = log_staged(h * (r2 * r2), h + h, p, tab);
                const double da = exp_neg_staged(-((0.5 * P.alpha) * lnd2), tab, cc);
                return h > 0x1p-999 ? da : 0.0;
            }
        }
        const double s = sqrt_lean(h);
        double p = 6435.0 / 557056.0;
        p = fma(p, h, 143.0 / 10240.0);
        p = fma(p, h, 231.0 / 13312.0);
        p = fma(p, h, 63.0 / 2816.0);
        p = fma(p, h, 35.0 / 1152.0);
        p = fma(p, h, 5.0 / 112.0);
        p = fma(p, h, 3.0 / 40.0);
        p = fma(p, h, 1.0 / 6.0);
        double d = r2 * fma(s * h, p, s);
        if constexpr (kc_family(KC) == 3) d = (P.alpha == 2.0) ? d * d : d;
        return d;
    } else {
        double d = dist_pos(xa - xb, ya - yb, cc);
        if constexpr (kc_family(KC) == 3) {
            if (P.alpha == 2.0) d = d * d;
            else if (P.alpha != 1.0) d = d > 0x1p-499 ? exp_neg_staged(-(P.alpha * log_staged(d, 0.0, 0.0, tab)), tab, cc) : 0.0;
        }
        return d;
    }
}

// The scaled distance r = da / beta of the closed forms, da = pair_dist_pow, at
// most 746: there e^-r is 0, and the powers of r that multiply it cannot bring
// it back (or overflow), however small beta is.  Kernels use this r in every
// factor.  A NaN becomes 746 as well, so callers validate their inputs.
__device__ __forceinline__ double scaled_dist(double da, double inv_beta, const CovConst &c) {
    return fmin(da * inv_beta, c.rmax);
}

// Covariance from r = scaled_dist and e = e^-r: sigma2 e^-r, sigma2 (1 + r) e^-r,
// sigma2 (1 + r + r^2 / 3) e^-r.  Every sum is an explicit
// FMA: kernels that share distances between parameter vectors must give the
// bits of those that do not, so nothing is left for the compiler to contract
// in one kernel and not in another.
template <int KC>
__device__ __forceinline__ double cov_value(double r, double e, const Params &P) {
    constexpr int F = kc_family(KC);
    if constexpr (F == 1) return fma(r, P.sigma2, P.sigma2) * e;
    else if constexpr (F == 2) return fma(r, fma(r, P.sigma2 * (1.0 / 3.0), P.sigma2), P.sigma2) * e;
    else return P.sigma2 * e;
}

// The beta-derivative of the covariance up to the pair-independent factor
// dbeta_scale: r e^-r, r^2 e^-r, (r^2 + r^3) e^-r.
template <int KC>
__device__ __forceinline__ double dbeta_raw(double r, double e) {
    constexpr int F = kc_family(KC);
    if constexpr (F == 1) return (r * r) * e;
    else if constexpr (F == 2) return fma(r * r, r, r * r) * e;
    else return r * e;
}
template <int KC>
__device__ __forceinline__ double dbeta_scale(const Params &P) {
    return (P.sigma2 * P.inv_beta) * (kc_family(KC) == 2 ? 1.0 / 3.0 : 1.0);
}

// Closed forms in the scaled distance r: Matern, Eq. (2), for half-integer
// smoothness (NU: 0 -> nu = 0.5, 1 -> nu = 1.5, 2 -> nu = 2.5, r = d / beta)
// and the power exponential (NU = 3, r = d^alpha / beta), whose form is the
// nu = 1/2 one.
template <int NU>
__device__ __forceinline__ double matern_r(double r, double sigma2) {
    double e = exp_neg(r);
    if constexpr (NU == 0 || NU == 3) {
        return sigma2 * e;
    } else if constexpr (NU == 1) {
        return sigma2 * ((1.0 + r) * e);
    } else {
        return sigma2 * ((1.0 + r * (1.0 + r * (1.0 / 3.0))) * e);
    }
}

// beta-derivative of the covariance: dC/dbeta = sigma2 h(r) / beta with
//   h = r e^-r (nu = 0.5), r^2 e^-r (nu = 1.5), r^2 (1 + r) e^-r / 3 (nu = 2.5).
template <int NU>
__device__ __forceinline__ double matern_dbeta_r(double r, double sigma2_over_beta) {
    double e = exp_neg(r);
    if constexpr (NU == 0 || NU == 3) {
        return sigma2_over_beta * (r * e);
    } else if constexpr (NU == 1) {
        return sigma2_over_beta * ((r * r) * e);
    } else {
        return sigma2_over_beta * ((r * r) * (1.0 + r) * (1.0 / 3.0) * e);
    }
}

__device__ __forceinline__ double dist2d(double ax, double ay, double bx, double by) {
    double dx = ax - bx;
    double dy = ay - by;
    return sqrt_dist(fma(dx, dx, dy * dy));
}

// 2^(j/64) as (hi, lo) pairs in global memory, for code that does not stage
// the table in LDS.
__device__ __forceinline__ const double *exp_table_global() { return reinterpret_cast<const double *>(kExp2Frac64); }

// Scaled distance of a pair under covariance code KC (the unblocked kernel's form).
template <int KC>
__device__ __forceinline__ double cov_r(double xa, double ya, double ca, double xb, double yb, double cb,
                                        const Params &P) {
    if constexpr (kc_gcd(KC)) {
        return cov_scaled<KC>(gcd_km(xa, ya, ca, xb, yb, cb), P, exp_table_global());
    } else {
        return cov_scaled<KC>(dist2d(xa, ya, xb, yb), P, exp_table_global());
    }
}

// Sum over the 64 lanes of a wavefront; fixed butterfly order, every lane gets the total.
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

// Block-wide sum in a fixed order.  `scratch` holds at least NWAVES doubles.
// Must be reached by every thread of the block.  Every thread gets the total.
template <int NWAVES>
__device__ __forceinline__ double block_sum(double v, double *scratch) {
    v = wave_sum(v);
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) scratch[wave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) t += scratch[w];
    return t;
}

// Double-double accumulation (Knuth two-sum), used for the final reductions.
struct DD {
    double hi, lo;
};

__device__ __forceinline__ DD dd_add(DD a, double b) {
    double s = a.hi + b;
    double bb = s - a.hi;
    double err = (a.hi - (s - bb)) + (b - bb);
    DD r;
    r.hi = s;
    r.lo = a.lo + err;
    double t = r.hi + r.lo;
    r.lo = r.lo - (t - r.hi);
    r.hi = t;
    return r;
}

__device__ __forceinline__ DD dd_add(DD a, DD b) {
    DD r = dd_add(a, b.hi);
    return dd_add(r, b.lo);
}

}  // namespace vecchia
