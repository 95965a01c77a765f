// rt_functions.h -- where a right-hand side takes its functions of one
// variable from (sin and cos of theta, the mass function F and dF/dR): a
// policy argument of rhs_c and attempt (rt_ray.h).
//
//   Direct   the functions of rt_math.h and rt_device.h as they stand.  Their
//            coefficients are literals, which the compiler materialises by
//            scalar moves beside each use: 362 s_mov_b32 among the 1381
//            instructions of a cored-NFW step attempt.
//   Pinned   the same arithmetic, operation for operation (the same bits), on
//            coefficients that the kernel loads into vector registers once.
//
// A wavefront alone on its SIMD issues an instruction every 2.0 ns (4.9 cycles at 2.4
// GHz) whatever its type, so the scalar moves are a quarter of its time; several
// wavefronts hide them behind each other's vector instructions, and three per
// SIMD hid most of them.  Pinned coefficients take 38 (Kerr), 64 (Einasto) or
// 76 (cored NFW) vector registers, so two wavefronts fit a SIMD instead of three:
// 239 to 253 registers in the trace kernels and no vector spills, and 1034
// instructions of the 1381 are left, 59 of them scalar moves (670 Kerr, 880 Einasto;
// counted between branches, as are all counts here).  The wide cored NFW (eta above
// 0.34) pins sine's and cosine's coefficients and 19 of the tableau's, not its
// logarithm's and exponential's: 211 scalar moves of 1256.  Measured
// with two pinned wavefronts against three that materialise (same bits, one
// launch, cored NFW chi = 0.94): 64^2 1.57 -> 1.25 ms, 256^2 1.56 -> 1.27,
// 512^2 2.36 -> 2.10, 1024^2 6.87 -> 6.72 ms; wide cored NFW (0.6, 8): 64^2 1.68 -> 1.54,
// 1024^2 8.25 -> 7.28; one pinned wavefront per SIMD is
// as fast up to 256^2 and 6 % slower at 1024^2.  So every binary64 kernel pins,
// at two wavefronts per SIMD, and no rule on the launch's size is needed.
//   Vector spills remain in Einasto's thick disc (four).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rt_device.h"
#include "rt_math.h"

namespace rt {
namespace fn {

// Dormand-Prince 5(4) tableau (Dormand & Prince 1980, first-same-as-last).
struct Tableau {
    double a21 = 0.2;
    double a31 = 3.0 / 40.0, a32 = 9.0 / 40.0;
    double a41 = 44.0 / 45.0, a42 = -56.0 / 15.0, a43 = 32.0 / 9.0;
    double a51 = 19372.0 / 6561.0, a52 = -25360.0 / 2187.0, a53 = 64448.0 / 6561.0, a54 = -212.0 / 729.0;
    double a61 = 9017.0 / 3168.0, a62 = -355.0 / 33.0, a63 = 46732.0 / 5247.0, a64 = 49.0 / 176.0,
           a65 = -5103.0 / 18656.0;
    double b1 = 35.0 / 384.0, b3 = 500.0 / 1113.0, b4 = 125.0 / 192.0, b5 = -2187.0 / 6784.0,
           b6 = 11.0 / 84.0;
    // error weights: 5th-order minus embedded 4th-order weights
    double e1 = 71.0 / 57600.0, e3 = -71.0 / 16695.0, e4 = 71.0 / 1920.0, e5 = -17253.0 / 339200.0,
           e6 = 22.0 / 525.0, e7 = -1.0 / 40.0;
};

struct Direct {};
__host__ __device__ __forceinline__ Tableau tableau(const Direct&) { return Tableau{}; }
template <class S>
__host__ __device__ __forceinline__ void sincos(const Direct&, const S& x, S* s_out, S* c_out) {
    dm::sincos(x, s_out, c_out);
}
// (sine and cosine up to a common sign: the right-hand side's products cancel it)
__host__ __device__ __forceinline__ void sincos(const Direct&, const double& x, double* s_out,
                                                double* c_out) {
    dm::sincos_pi(x, s_out, c_out);
}
template <int METRIC, class K, class S>
__host__ __device__ __forceinline__ void mass_function(const Direct&, const K& c, const S& R, S& F,
                                                       S& dF) {
    rt::mass_function<METRIC>(c, R, F, dF);
}

// The coefficients of dm::sincos_pi, dm::log_kernel, dm::expm1_near and dm::exp
// (highest degree first) with their reduction constants.
template <bool SCALAR>
struct PinnedSet {
    double s[8] = {2.7314447669863206e-15, -7.643970296798566e-13, 1.6058977312464087e-10,
                   -2.5052107616996182e-08, 2.7557319219163234e-06, -0.00019841269841254974,
                   0.008333333333333316, -0.16666666666666666};
    double c[8] = {4.627675985018022e-14, -1.1464689885720016e-11, 2.0876630867422994e-09,
                   -2.755731776732053e-07, 2.4801587292446213e-05, -0.0013888888888860709,
                   0.04166666666666634, -0.5};
    double inv_pi = dm::kInvPi, pi_hi = dm::kPiHi, pi_mid = dm::kPiMid;
    double lw[7] = {4.460586451734852e-06, 1.8715480469428627e-05, 8.878363830694202e-05,
                    0.0004340275612264664, 0.002232142861404335, 0.012499999999968595,
                    0.08333333333333337};
    double en[8] = {2.399505199127987e-07, 2.7335759431393298e-06, 2.4794062080910826e-05,
                    0.00019841120114754993, 0.001388888713436031, 0.00833333332176611,
                    0.041666666666284255, 0.1666666666666618};
    double ex[10] = {2.091467937680297e-09, 2.5105206374263736e-08, 2.755727366134811e-07,
                     2.75572554257457e-06, 2.4801587325533363e-05, 0.00019841269874800493,
                     0.0013888888888883752, 0.008333333333326141, 0.04166666666666667,
                     0.1666666666666667};
    double ln2_hi = dm::kLn2Hi, ln2_lo = dm::kLn2Lo, inv_ln2 = dm::kInvLn2;
    Tableau rk;
};
template <bool S>
__host__ __device__ __forceinline__ const Tableau& tableau(const PinnedSet<S>& q) {
    return q.rk;
}
using Pinned = PinnedSet<false>;
// The thick disc's kernel has registers for sine's and cosine's coefficients
// only; those of its exponentials and logarithm go through scalar registers at
// each use (left to itself the compiler builds them in vector registers, two
// vector moves a coefficient).
using PinnedThick = PinnedSet<true>;

// The coefficients as the kernel of a metric holds them: in vector registers,
// opaque to the compiler so that it cannot turn them back into literals.
constexpr int kAll = -1;   // every metric's coefficients (the batched kernel)
template <int METRIC, bool SCALAR = false>
__device__ __forceinline__ PinnedSet<SCALAR> pin() {
    PinnedSet<SCALAR> p;
#if defined(__HIP_DEVICE_COMPILE__)
    auto hold = [](double& x) { asm volatile("" : "+v"(x)); };
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        hold(p.s[i]);
        hold(p.c[i]);
    }
    hold(p.s[7]);
    hold(p.inv_pi);
    hold(p.pi_hi);
    hold(p.pi_mid);
    if constexpr (!SCALAR && (METRIC == CNFW_NEAR || METRIC == kAll)) {
#pragma unroll
        for (int i = 0; i < 7; ++i) hold(p.lw[i]);
#pragma unroll
        for (int i = 0; i < 8; ++i) hold(p.en[i]);
        hold(p.ln2_hi);
        hold(p.ln2_lo);
    }
    if constexpr (!SCALAR && METRIC == EINASTO) {
#pragma unroll
        for (int i = 0; i < 10; ++i) hold(p.ex[i]);
        hold(p.ln2_hi);
        hold(p.ln2_lo);
        hold(p.inv_ln2);
    }
    // and as many of the tableau's as every kernel has registers left for without
    // a spill (the gradient's forward pass is the fullest).  Kerr 64^2 772 -> 744
    // us, 512^2 1423 -> 1383; Einasto 64^2 883 -> 851; no difference at 1024^2,
    // where two wavefronts hide the scalar moves, nor for seven in the cored NFW.
    constexpr int n = SCALAR || METRIC == kAll ? 0
                      : METRIC == KERR         ? 23
                      : METRIC == EINASTO      ? 10
                      : METRIC == CNFW_NEAR    ? 0
                                               : 19;
    double* const rk[] = {&p.rk.a61, &p.rk.a62, &p.rk.a63, &p.rk.a64, &p.rk.a65, &p.rk.a51, &p.rk.a52,
                          &p.rk.a53, &p.rk.a54, &p.rk.a41, &p.rk.a42, &p.rk.a43, &p.rk.a31, &p.rk.a32,
                          &p.rk.b1,  &p.rk.b3,  &p.rk.b4,  &p.rk.b5,  &p.rk.b6,  &p.rk.e1,  &p.rk.e3,
                          &p.rk.e4,  &p.rk.e5,  &p.rk.e6,  &p.rk.e7,  &p.rk.a21};
#pragma unroll
    for (int i = 0; i < n; ++i) hold(*rk[i]);
#endif
    return p;
}

template <bool SCALAR = false, int N>
__host__ __device__ __forceinline__ double horner(const double (&c)[N], double x) {
    double p = c[0];
#pragma unroll
    for (int i = 1; i < N; ++i) {
        double ci = c[i];
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (SCALAR) asm("" : "+s"(ci) : "v"(p));
#endif
        p = fma(p, x, ci);
    }
    return p;
}

template <bool S>
__host__ __device__ __forceinline__ int32_t sincos_pi(const PinnedSet<S>& q, double x, double* s_out,
                                                      double* c_out) {
    const dm::NearestInt n = dm::nearest_int(x, q.inv_pi);
    double r = fma(-n.k, q.pi_hi, x);
    r = fma(-n.k, q.pi_mid, r);
    const double z = r * r;
    *s_out = fma(r * z, horner(q.s, z), r);
    *c_out = fma(z, horner(q.c, z), 1.0);
    return n.i;
}

template <bool S>
__host__ __device__ __forceinline__ void sincos(const PinnedSet<S>& q, const double& x, double* s_out,
                                                double* c_out) {
    sincos_pi(q, x, s_out, c_out);
}

// With their signs (the thick disc's source needs them).
__host__ __device__ __forceinline__ void signed_sincos(const Direct&, double x, double* s_out,
                                                       double* c_out) {
    dm::sincos(x, s_out, c_out);
}
template <bool S>
__host__ __device__ __forceinline__ void signed_sincos(const PinnedSet<S>& q, double x, double* s_out,
                                                       double* c_out) {
    const int32_t k = sincos_pi(q, x, s_out, c_out);
    dm::flip_signs(k, s_out, c_out);
}

// e^x and log(1 + u), as dm::exp and dm::log1p.
__host__ __device__ __forceinline__ double exp(const Direct&, double x) { return dm::exp(x); }
__host__ __device__ __forceinline__ double log1p(const Direct&, double u) { return dm::log1p(u); }
template <bool S>
__host__ __device__ __forceinline__ double exp(const PinnedSet<S>& q, double x) {
    const double xc = fmin(fmax(x, -760.0), 720.0);
    const dm::NearestInt n = dm::nearest_int(xc, q.inv_ln2);
    double r = fma(-n.k, q.ln2_hi, xc);
    r = fma(-n.k, q.ln2_lo, r);
    const double p = fma(horner<S>(q.ex, r), r, 0.5);
    return ldexp(1.0 + fma(r * r, p, r), n.i);
}
template <bool S>
__host__ __device__ __forceinline__ double log1p(const PinnedSet<S>& q, double u) {
    const double v = 1.0 + u;
#if defined(__HIP_DEVICE_COMPILE__)
    const double corr = (u - (v - 1.0)) * __builtin_amdgcn_rcp(v);
#else
    const double corr = (u - (v - 1.0)) / v;
#endif
    int e;
    double m = frexp(v, &e);
    if (m < 0.70710678118654752) {
        m *= 2.0;
        e -= 1;
    }
    const double w = fma(m, 2.0, -2.0) * dm::recip(m + 1.0);
    const double z = w * w;
    const double logm = fma(w * z, horner<S>(q.lw, z), w);
    const double de = static_cast<double>(e);
    return fma(de, q.ln2_hi, logm + fma(de, q.ln2_lo, corr));
}

template <int METRIC, class K, bool S>
__host__ __device__ __forceinline__ void mass_function(const PinnedSet<S>& q, const K& c, const double& R,
                                                       double& F, double& dF) {
    if constexpr (METRIC == EINASTO) {
        const double x = R * c.inv_lam;
        const double e = exp(q, -x);
        const double mu = 1.0 - e * (1.0 + x * (1.0 + 0.5 * x));
        const double dmu = 0.5 * e * x * x * c.inv_lam;
        F = 2.0 * R * mu;
        dF = 2.0 * (mu + R * dmu);
    } else if constexpr (METRIC == CNFW_NEAR) {
        const double Rl = R + c.lam_c;
        const dm::LogSplit s = dm::log_split(fma(R, c.inv_lam_c, 1.0));
        const double d = R * Rl;
        const double inv = dm::recip1(fma(d, s.m, d));
        const double a = fma(s.m, inv, inv);
        const double iR = Rl * a, iRl = R * a;
        const double w = fma(s.m, 2.0, -2.0) * (d * inv);
        const double v = w * w;
        const double lk = fma(w * v, horner<S>(q.lw, v), w);
        const double lg = fma(s.e, q.ln2_hi, fma(s.e, q.ln2_lo, lk));
        const double ex = c.eta_lc * (iRl - 2.0 * iR * lg);
        const double dex = c.eta_lc * (2.0 * iR * (iR * lg - iRl) - iRl * iRl);
        const double em1 = fma(ex * ex, fma(horner<S>(q.en, ex), ex, 0.5), ex);
        F = R * (2.0 - R * em1);
        dF = 2.0 - R * (2.0 * em1 + R * (em1 + 1.0) * dex);
    } else {
        rt::mass_function<METRIC>(c, R, F, dF);
    }
}

}  // namespace fn
}  // namespace rt
