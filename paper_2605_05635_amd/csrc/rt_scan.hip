// rt_scan.hip -- parameter scans of the spacetimes (Sec. 2): per point, the
// outer horizon (eq. (33)), the ergosurface radius at one polar angle, and the
// extremal spin with its radius.  One wavefront per point, with the results of
// rt_scan.h's serial searches to the bit: the same grid edges, the interval the
// serial search would have kept, the same bisection.
//
// What bounds it is the count of F(R) evaluations, each about 150 binary64
// instructions: the serial searches make 60,000 per point.  Nearly all of them
// ask about intervals that cannot matter, and that can be known from a few:
// q(R) = F/R, twice the enclosed mass, does not fall with R in any of the three
// spacetimes (Kerr: constant; Einasto: mu' > 0; cored NFW with eta >= 0: with u
// the negative exponent, (R u)' = eta lambda_c (2 R + lambda_c)/(R + lambda_c)^2
// > 0, hence u + R u' > 0 and q' = 1 - e^-u + R u' e^-u >= e^-u (u + R u') > 0).  So on
// lo <= R <= hi
//     R^2 - F >= R^2 - q(hi) R,    2 R - F' <= 2 hi - q(lo),
// and 64 samples of q rule out, with a margin far above rounding, the
// intervals in which R^2 - F + a2 is positive (no root) or above a value already
// sampled (not the least minimum) or in which it falls (no minimum).  What is left, some
// hundred grid intervals, is evaluated one per lane, and bisections evaluate the
// next four halvings' 15 midpoints at once, for three searches side by side.
// 4096 points of the cored NFW: 796 -> 29 us; the results' bits, NaNs included,
// are those of the evaluation of every interval.
#include "rt.h"
#include "rt_device.h"

namespace rt {
namespace {

// Grid intervals k = 1..n of the two serial searches, by their own loop
// conditions, counted at compile time.  (Counted on the device, the 59,986
// dependent add-and-compare steps took three quarters of the kernel.)
constexpr int root_intervals() {
    int n = 0;
    while (50.0 - (n + 1) * 1e-2 >= 0.05 - 1e-12) ++n;
    return n;
}
constexpr int spin_intervals() {
    int n = 0;
    while (0.01 + static_cast<double>(n) * 1e-3 < 50.0) ++n;
    return n;
}
constexpr int kRootIntervals = root_intervals(), kSpinIntervals = spin_intervals();

// scan::delta for one spacetime.
template <int METRIC>
__device__ __forceinline__ void delta(const ImageConst& c, double a2, double R, double* D,
                                      double* dD) {
    double F, dF;
    mass_function<METRIC>(c, R, F, dF);
    *D = R * R - F + a2;
    *dD = 2.0 * R - dF;
}

// Edge k of the two grids.
__device__ __forceinline__ double root_edge(int k) {
    const double top = 50.0, step = 1e-2;
    return top - k * step;
}
__device__ __forceinline__ double spin_edge(int k) {
    const double step = 1e-3;
    return 0.01 + static_cast<double>(k) * step;
}

// R^2 - F + a2 is above `least` on all of [lo, hi]: with q = q(hi), by a margin
// above the rounding of F (relative 1e-15, and the cored NFW's logarithm, exact
// to 2e-16, times 2 eta lambda_c R).  False for NaN and infinities.
__device__ __forceinline__ bool above(const ImageConst& c, double lo, double hi, double q, double a2,
                                      double least) {
    const double margin = 1e-6 * (hi * hi + q * hi + a2) + 1e-12 * c.eta_lc * hi;
    const double h = 0.5 * q;
    const double low = lo >= h ? lo * (lo - q) : -h * h;
    return low + a2 - margin > least;
}

// R^2 - F falls on all of [lo, hi], with q = q(lo).
__device__ __forceinline__ bool falls(const ImageConst& c, double hi, double q) {
    return 2.0 * hi + 1e-6 * (hi + q) + 1e-12 * c.eta_lc < q;
}

// Bisection to the last representable bracket, as the serial searches do it
// (200 halvings at most): [a, b] becomes the half whose lower end still has
// D <= 0 (`slope`: D' < 0).  2^LEVELS lanes per bracket evaluate the midpoints
// of its next LEVELS halvings, lane i node i of their tree, and follow the path.
template <int METRIC, int LEVELS>
__device__ void bisect(const ImageConst& c, double a2, bool slope, bool open, double& a, double& b) {
    constexpr int kLanes = 1 << LEVELS;
    const int lane = __lane_id(), node = lane % kLanes > 0 ? lane % kLanes : 1;
    const int depth = 31 - __clz(node);
    int left = 200;
    while (__any(open)) {
        double u = a, v = b;
#pragma unroll
        for (int s = LEVELS - 2; s >= 0; --s) {
            const double m = 0.5 * (u + v);
            if (s < depth) {
                if (node >> s & 1) u = m; else v = m;
            }
        }
        double D, dD;
        delta<METRIC>(c, a2, 0.5 * (u + v), &D, &dD);
        const unsigned long long up = __ballot(slope ? dD < 0.0 : !(D > 0.0)) >> (lane & ~(kLanes - 1));
        int at = 1;
#pragma unroll
        for (int s = 0; s < LEVELS; ++s) {
            const double m = 0.5 * (a + b);
            open = open && left > 0 && !(m <= a || m >= b);
            if (open) {
                const int bit = static_cast<int>(up >> at & 1);
                if (bit) a = m; else b = m;
                at = 2 * at + bit;
                --left;
            }
        }
    }
}

// The bracket that the serial largest_root bisects.  R and q = F/R are this
// lane's coarse edge, 80 grid intervals apart; D_top is D at the top.
constexpr int kRootCoarse = (kRootIntervals + 62) / 63;
template <int METRIC>
__device__ bool root_bracket(const ImageConst& c, double a2, double R, double q, double* a, double* b) {
    const int lane = __lane_id();
    const double Rhi = __shfl_up(R, 1), qhi = __shfl_up(q, 1);
    const unsigned long long keep = __ballot(lane > 0 && !above(c, R, Rhi, qhi, a2, 0.0));
    if (keep == 0ull) return false;
    const int first = __ffsll(static_cast<long long>(keep)) - 1, last = 63 - __clzll(keep);
    const int end = last * kRootCoarse < kRootIntervals ? last * kRootCoarse : kRootIntervals;
    for (int k0 = (first - 1) * kRootCoarse; k0 < end; k0 += 63) {
        const int k = k0 + lane;
        double D, dD;
        delta<METRIC>(c, a2, root_edge(k < end ? k : end), &D, &dD);
        const double dD_hi = __shfl_up(dD, 1);
        unsigned long long some =
            __ballot(lane > 0 && k <= end && (D <= 0.0 || (dD < 0.0 && dD_hi > 0.0)));
        for (; some != 0ull; some &= some - 1) {   // from the top
            const int src = __ffsll(static_cast<long long>(some)) - 1;
            *a = root_edge(k0 + src);
            *b = root_edge(k0 + src - 1);
            if (__shfl(D, src) <= 0.0) return true;
            // interior minimum: located where the derivative vanishes
            double u = *a, v = *b, Dm, dDm;
            bisect<METRIC, 6>(c, a2, true, true, u, v);
            *a = 0.5 * (u + v);
            delta<METRIC>(c, a2, *a, &Dm, &dDm);
            if (Dm <= 0.0) return true;
        }
    }
    return false;
}

// The least minimum of R^2 - F so far, and an interval with a minimum that has
// not been located yet (the last one is, together with the roots).
struct Minimum {
    double best = 0.0, best_r = 0.0, lo = 0.0, hi = 0.0;
    bool found = false, pending = false;
};

template <int METRIC>
__device__ void settle(const ImageConst& c, Minimum& m) {
    const double r = 0.5 * (m.lo + m.hi);
    double V, dV;
    delta<METRIC>(c, 0.0, r, &V, &dV);
    if (V < m.best) {
        m.best = V;
        m.best_r = r;
        m.found = true;
    }
    m.pending = false;
}

// Intervals begin + 1..end of the extremal-spin grid, in the serial order.
template <int METRIC>
__device__ void sweep(const ImageConst& c, int begin, int end, Minimum& m) {
    const int lane = __lane_id();
    for (int k0 = begin; k0 < end; k0 += 63) {
        const int k = k0 + lane;
        double V, dV;
        delta<METRIC>(c, 0.0, spin_edge(k < end ? k : end), &V, &dV);
        const double dV_lo = __shfl_up(dV, 1);
        unsigned long long some = __ballot(lane > 0 && k <= end && dV_lo < 0.0 && dV >= 0.0);
        for (; some != 0ull; some &= some - 1) {
            if (m.pending) {
                bisect<METRIC, 6>(c, 0.0, true, true, m.lo, m.hi);
                settle<METRIC>(c, m);
            }
            const int src = __ffsll(static_cast<long long>(some)) - 1;
            m.lo = spin_edge(k0 + src - 1);
            m.hi = spin_edge(k0 + src);
            m.pending = true;
        }
    }
}

// Horizon, ergosurface radius, extremal spin and its radius (NaN: none).
template <int METRIC>
__device__ void search(const ImageConst& c, double a2_ergo, double* res) {
    const int lane = __lane_id();
    bool has[2];
    double a[2], b[2];
    const double a2[2] = {c.chi2, a2_ergo};
    {
        const int k = lane * kRootCoarse < kRootIntervals ? lane * kRootCoarse : kRootIntervals;
        const double R = root_edge(k);
        double F, dF;
        mass_function<METRIC>(c, R, F, dF);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = b[i] = 0.0;
            has[i] = __shfl(R * R - F + a2[i], 0) > 0.0 &&
                     root_bracket<METRIC>(c, a2[i], R, F / R, &a[i], &b[i]);
        }
    }

    // The extremal spin's minimum: the intervals that can hold the least one,
    // narrowed twice.  A minimum counts below 0 only, and when some sample is
    // below 0 the least one can be expected to be no higher than it; where the
    // minima found are (the sample was next to an end of the grid), all are.
    int begin = 0, end = kSpinIntervals;
    double least = 0.0;
#pragma unroll
    for (int stage = 0; stage < 2 && begin < end; ++stage) {
        const int per = (end - begin + 62) / 63, k = begin + lane * per;
        const double R = spin_edge(k < end ? k : end);
        double F, dF;
        mass_function<METRIC>(c, R, F, dF);
        const double q = F / R;
        double v = R * R - F + 1e-9;   // (a minimum is below its sample but for rounding)
        for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
        least = fmin(least, v);
        const double Rlo = __shfl_up(R, 1), qlo = __shfl_up(q, 1);
        const unsigned long long keep =
            __ballot(lane > 0 && !above(c, Rlo, R, q, 0.0, least) && !falls(c, R, qlo));
        const int from = begin;
        begin = keep ? from + (__ffsll(static_cast<long long>(keep)) - 2) * per : end;
        const int to = from + (63 - __clzll(keep | 1ull)) * per;
        end = to < end ? to : end;
    }
    Minimum m;
    sweep<METRIC>(c, begin, end, m);

    // lanes 0-15 the horizon, 16-31 the ergosurface, 32-47 the pending minimum
    const int job = lane / 16;
    double u = job == 0 ? a[0] : job == 1 ? a[1] : m.lo, v = job == 0 ? b[0] : job == 1 ? b[1] : m.hi;
    bisect<METRIC, 4>(c, job == 0 ? a2[0] : job == 1 ? a2[1] : 0.0, job == 2,
                      job == 0 ? has[0] : job == 1 ? has[1] : job == 2 && m.pending, u, v);
    const double r = 0.5 * (u + v);
    if (has[0]) res[0] = __shfl(r, 0);
    if (has[1]) res[1] = __shfl(r, 16);
    if (m.pending) {
        m.lo = __shfl(u, 32);
        m.hi = __shfl(v, 32);
        settle<METRIC>(c, m);
    }
    if (least < 0.0 && !(m.found && m.best <= least)) {
        m = Minimum{};
        sweep<METRIC>(c, 0, kSpinIntervals, m);
        if (m.pending) {
            bisect<METRIC, 6>(c, 0.0, true, true, m.lo, m.hi);
            settle<METRIC>(c, m);
        }
    }
    if (m.found) {
        res[2] = sqrt(-m.best);
        res[3] = m.best_r;
    }
}

__global__ __launch_bounds__(256) void scan_kernel(const rt_scan_point* __restrict__ pts, int32_t n,
                                                   double* __restrict__ out) {
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / 64;
    if (i >= n) return;   // whole wavefronts
    const rt_scan_point q = pts[i];
    const double nan = __builtin_nan("");
    double res[4] = {nan, nan, nan, nan};
    const bool ok_metric = q.metric == RT_KERR ||
                           (q.metric == RT_EINASTO && q.halo[0] > 0.0) ||
                           (q.metric == RT_CNFW && q.halo[0] >= 0.0 && q.halo[1] > 0.0);
    if (ok_metric && q.reserved == 0 && isfinite(q.spin) && isfinite(q.theta) &&
        isfinite(q.halo[0]) && isfinite(q.halo[1])) {
        ImageConst c{};
        c.metric = q.metric;
        c.chi = q.spin;
        c.chi2 = q.spin * q.spin;
        if (q.metric == RT_EINASTO) c.inv_lam = 1.0 / q.halo[0];
        if (q.metric == RT_CNFW) {
            c.lam_c = q.halo[1];
            c.inv_lam_c = 1.0 / q.halo[1];
            c.eta_lc = q.halo[0] * q.halo[1];
        }
        const double co = cos(q.theta);
        const double a2_ergo = c.chi2 * co * co;
        if (q.metric == RT_KERR)
            search<KERR>(c, a2_ergo, res);
        else if (q.metric == RT_EINASTO)
            search<EINASTO>(c, a2_ergo, res);
        else
            search<CNFW>(c, a2_ergo, res);
    }
    if (__lane_id() == 0)
        for (int j = 0; j < 4; ++j) out[4 * i + j] = res[j];
}

}  // namespace

hipError_t launch_scan(const ::rt_scan_point* pts, int32_t n, double* out, hipStream_t stream) {
    const int64_t threads = static_cast<int64_t>(n) * 64;
    hipLaunchKernelGGL(scan_kernel, dim3(static_cast<uint32_t>((threads + 255) / 256)), dim3(256), 0,
                       stream, pts, n, out);
    return hipGetLastError();
}

}  // namespace rt
