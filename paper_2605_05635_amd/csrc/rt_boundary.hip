// rt_boundary.hip -- gfx950 kernel of the shadow-boundary search (Sec. 4.1,
// eqs. (78)-(79)): along a screen direction (cos psi, sin psi), the impact
// parameter b at which the rays from X = b cos psi, Y = b sin psi turn from
// captured to escaping.  A wavefront holds 64 / S directions, S lanes each
// (S = 64, 32 or 16 samples per pass), and a pass traces one ray per lane.
//
// The result is defined by multisection: level 1 divides the bracket into S + 1
// cells and keeps the one below the first escaping edge, level 2 divides that
// one, and so on until a cell is no wider than b_tol.  A pass that samples the S
// inner edges of one level gains that level (a uniform pass).  Every ray of a
// late pass winds around the photon shell, so passes are what costs: nine of
// them at S = 16 from 7 M to 1e-10 M, the last of rays of up to 1716 attempts
// near the polar axis, one after another.  A guided pass samples edges two or
// three levels down, around a prediction of the transition, and gains those
// levels at once when it holds; the cell kept is always one whose two edges
// have been traced, so the brackets are multisection's where the fates are in
// order (kGuidedTol, redo below).
//
// The prediction: near the unstable orbit a ray's radial time tau = int dlambda
// / Sigma (which the polar motion does not enter) diverges as -a ln|b - b_c|
// with the same a on both sides.  Two escaping and two captured samples next to
// the transition give a and b_c.  The error left, in units of the bracket W
// that held the samples, is of second order, about W/2 until W ~ 1e-3, and
// below 1e-4 from there (measured over 12 directions of the cored-NFW and Kerr
// holes); without Sigma in the clock it stays at 2e-2.
//
// Directions advance independently, each from pass to pass as soon as its own
// rays end.  4096 directions at S = 16, cored NFW chi = 0.94: 23.0 -> 15.1
// ms (five to seven passes in place of nine); 1000 at S = 64: 12.6 -> 8.3 ms.
// What is left is the longest direction's chain, 5924 attempts of 2.4 us; 20
// ms in one call of ten, where some direction came out of order (redo).
#include "rt_ray.h"

namespace rt {
namespace {

using namespace ray;

constexpr int kMaxLevels = 64;
// Looser integrations search by uniform passes.  Fates are out of order within the
// integration's error of the transition, where an accept or reject decision flips
// between neighbouring rays, and samples that a guided pass leaves out can
// then miss a flip: with guided passes at every tolerance the bracket was another
// one for none of 184,320 directions at 1e-8 (S = 16) and of 98,304 at 1e-7, for 17 of
// 86,016 at 1e-6 and for 71 of 19,400 from 1e-5 to 1e-2 (one in 17 from 1e-6 to
// 1e-2 without the test of order in redo below).
constexpr double kGuidedTol = 1e-7;
constexpr int kMay = 1, kDid = 2;   // a direction may run guided passes, has run one
// The prediction lies above the transition by 0.2 W to 0.75 W of the bracket W
// (the sides' next order); taking off 0.45 W settles 4096 directions at S = 16 in
// five passes for 3294 of them and in six or seven for the others, against 2823
// without it (0.25: 3143, 0.7: 3120; the same order in four other spacetimes).
constexpr double kBias = 0.45;

// What a direction keeps between passes: its two nearest escaping samples with
// their radial times (b_c < e1 < e2; infinity where there is none), and its two
// nearest captured ones (c2 < c1 < b_c; minus infinity).  In LDS, one per
// direction of the workgroup, written alike by all its lanes.
struct Nearest {
    double e1, te1, e2, te2, c1, tc1, c2, tc2;
    double lo, hi;   // the bracket
};

// Edge j of cell division (lo, hi, w), j = 0..S + 1 (no contraction: every use
// gives the same bits).
__device__ __forceinline__ double edge(double lo, double hi, double w, int j, int S) {
    if (j <= 0) return lo;
    if (j > S) return hi;
    const double t = static_cast<double>(j) * w;
    return lo + t;
}

// Cell j = 1..S + 1 of (lo, hi, w).
__device__ __forceinline__ void cell(double& lo, double& hi, double w, int j, int S) {
    const double nlo = edge(lo, hi, w, j - 1, S), nhi = edge(lo, hi, w, j, S);
    lo = nlo;
    hi = nhi;
}

// The smallest (largest) of v over the S lanes of a group, with the t of a lane
// that has it.
__device__ __forceinline__ void group_min(double& v, double& t, int S) {
    for (int off = 1; off < S; off <<= 1) {
        const double v2 = __shfl_xor(v, off), t2 = __shfl_xor(t, off);
        if (v2 < v) {
            v = v2;
            t = t2;
        }
    }
}

// Takes sample (v, t) into the ordered pair (a, ta), (b, tb), a < b.
__device__ __forceinline__ void keep_two(double v, double t, volatile double& a, volatile double& ta,
                                         volatile double& b, volatile double& tb) {
    if (v < a) {
        b = a;
        tb = ta;
        a = v;
        ta = t;
    } else if (v > a && v < b) {
        b = v;
        tb = t;
    }
}

// The transition predicted from n: x in (c1, e1) where the two sides' logarithmic
// slopes agree, by bisection.  False without four finite samples that diverge
// towards the transition.
__device__ __forceinline__ bool predict(const volatile Nearest& n, double* x_out) {
    const double c1 = n.c1, c2 = n.c2, e1 = n.e1, e2 = n.e2;
    const double De = n.te1 - n.te2, Dc = n.tc1 - n.tc2;
    if (!(c2 > -INFINITY && e2 < INFINITY && De > 0.0 && Dc > 0.0 && De < INFINITY && Dc < INFINITY))
        return false;
    double a = c1, b = e1;
    for (int it = 0; it < 32; ++it) {
        const double x = 0.5 * (a + b);
        const float fe = __builtin_amdgcn_logf(static_cast<float>((e2 - x) * dm::recip1(e1 - x)));
        const float fc = __builtin_amdgcn_logf(static_cast<float>((x - c2) * dm::recip1(x - c1)));
        if (De * fc > Dc * fe) a = x; else b = x;
    }
    *x_out = 0.5 * (a + b);
    return true;
}

// Register-allocated like the trace kernel.
template <int METRIC>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void boundary_kernel(
    ImageConst c, const double* __restrict__ dirs, int32_t n, int32_t S, double b_lo, double b_hi,
    double b_tol, double* __restrict__ out, int32_t* __restrict__ status,
    int64_t* __restrict__ attempts) {
    __shared__ Nearest kept[kBlock / 16];
    const int64_t wave = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) / 64;
    const int lane = __lane_id();
    const int G = 64 / S;                    // directions per wavefront
    const int grp = lane / S, sl = lane - grp * S;
    const int64_t dir = wave * G + grp;
    const unsigned long long gmask = S == 64 ? ~0ull : ((1ull << S) - 1ull);
    const fn::Pinned fns = fn::pin<METRIC, false, false>();
    const Hot k = hot_of(c);
    const OutPtrs none{};    // no per-pixel outputs
    const bool mine = dir < n;
    volatile Nearest& near = kept[(threadIdx.x / 64) * 4 + grp];
    near.e1 = near.e2 = INFINITY;
    near.c1 = near.c2 = -INFINITY;
    near.te1 = near.te2 = near.tc1 = near.tc2 = 0.0;
    near.lo = b_lo;
    near.hi = b_hi;
    int64_t used = 0;        // this lane's step attempts
    int32_t result = 1;      // bracket without the transition, until checked
    bool done = !mine;
    // A caller that counts attempts gets the count of uniform passes.
    bool guided = false;     // the next pass (group-uniform)
    int guide = attempts == nullptr && fmax(c.rtol, c.atol) <= kGuidedTol ? kMay : 0;
    // Pass -1 checks the bracket (sample 0 at b_lo must stay inside, sample 1
    // at b_hi must escape); the passes after it search.  Each group runs its
    // passes on its own: when the last of its rays ends it narrows its bracket
    // and starts its next pass at once, while the other groups' rays are still
    // in flight.
    int level = -1;          // levels of the multisection done (-1: bracket unchecked)
    Ray r;
    double b = 0.0, tau = 0.0;   // this lane's sample and its radial time
    bool active = false;     // this lane's ray is in flight
    bool traced = false;     // it has one in the group's current pass,
    int32_t fate = 0;        // which ended so
    // Guided passes stop at cells of this width: below it rounding may decide
    // single rays' fates, and the levels left go edge by edge from the first.
    const double finest = fmax(b_tol, 1e-11 * b_hi);
    auto start_pass = [&]() {
        const double lo = near.lo, hi = near.hi;
        const double w = (hi - lo) / (S + 1);
        double x = 0.0;
        traced = true;
        if (level < 0) {
            b = sl == 0 ? b_lo : b_hi;
            traced = sl < 2;
        } else {
            // The finest level, at most three down, whose cells the prediction
            // is expected to miss by no more than S / 4.
            const double miss = 0.5 * (hi - lo) + 3e-4;   // in units of the bracket
            int m = 1;
            double cells = miss * (S + 1);
            while (m < 3 && cells * (S + 1) <= 0.25 * S) {
                ++m;
                cells *= S + 1;
            }
            if (guided && m > 1 && w > finest && predict(near, &x)) {
                guide |= kDid;
                // The S - S/4 edges of that level (or of the last before b_tol)
                // nearest to the prediction, and S/4 of the level above in
                // case it misses by more.
                x = fmax(x - kBias * (hi - lo) * (hi - lo), lo);
                const int coarse = S / 4;
                const bool fine = sl >= coarse;
                const int target = fine ? m : m - 1;
                double l = lo, h = hi, lw = w;
                int j = 0, at = 1;
                for (;; ++at) {
                    lw = (h - l) / (S + 1);
                    const double q = (x - l) / lw;
                    j = q >= static_cast<double>(S) ? S + 1 : static_cast<int>(q) + 1;
                    if (j < 1) j = 1;
                    if (at >= target) break;
                    double nl = l, nh = h;
                    cell(nl, nh, lw, j, S);
                    if (!(nh - nl > finest)) break;   // the last level
                    l = nl;
                    h = nh;
                }
                const int idx = fine ? j - (S - coarse) / 2 + (sl - coarse) : j - coarse / 2 + sl;
                traced = idx >= 1 && idx <= S && (fine || at == target);
                b = edge(l, h, lw, idx, S);
            } else {
                b = edge(lo, hi, w, sl + 1, S);
            }
        }
        active = traced;
        fate = 0;
        if (active)
            start_ray_dir<METRIC>(c, k, screen_dir_xy(c, b * dirs[2 * dir], b * dirs[2 * dir + 1]), 0, r, fns);
    };
    // Whether this pass's samples are dropped.  The edges that guided passes leave
    // out do not matter as long as fates are in order, captured below the
    // transition and escaping above.  A sample that ended inside above one that
    // escaped is out of order: the direction goes on by uniform passes from the
    // bracket that it had.  (Below `finest` they are uniform in any case.)  A ray
    // that ran out of attempts or whose error estimate was not finite counts as
    // inside on either side: from the start by uniform passes.
    auto redo = [&]() {
        double out_b = traced && fate == RAY_ESCAPED ? b : INFINITY, t = 0.0;
        group_min(out_b, t, S);
        out_b = fmin(out_b, near.e1);
        const bool lost = fate != 0 && fate != RAY_ESCAPED && fate != RAY_CAPTURED;
        const bool order = near.hi - near.lo > finest &&
                           (near.c1 > out_b || (traced && fate != RAY_ESCAPED && b > out_b));
        int odd = lost ? 2 : order ? 1 : 0;
        for (int off = 1; off < S; off <<= 1) odd |= __shfl_xor(odd, off);
        if (odd == 0 || !(guide & kMay)) return false;
        const bool drop = guide & kDid;
        guide = 0;
        if (drop && (odd & 2)) {
            near.e1 = near.e2 = INFINITY;
            near.c1 = near.c2 = -INFINITY;
            near.lo = b_lo;
            near.hi = b_hi;
            level = 0;
        }
        return drop;
    };
    if (!done) start_pass();
    while (__ballot(!done) != 0ull) {
        if (active) {
            const int32_t st = attempt<METRIC, StageNone, false, fn::Pinned, true>(k, none, 0, r, StageNone{}, fns);
            if (st != 0) {
                active = false;
                fate = st;
                // the radial time at the stop radius itself
                const double stop = st == RAY_ESCAPED ? k.r_esc : k.r_stop;
                tau = r.tau + (stop - r.y[1]) * (r.iS / r.k1[1]);
                used += r.attempts;
            }
        }
        const unsigned long long busy = (__ballot(active) >> (grp * S)) & gmask;
        const unsigned long long esc = (__ballot(fate == RAY_ESCAPED) >> (grp * S)) & gmask;
        if (!done && busy == 0ull) {
            // the group's pass is complete
            if (level < 0) {
                if ((esc & 1ull) || !(esc & 2ull)) {
                    done = true;
                } else {
                    result = 0;
                }
                level = 0;
                if (!(b_hi - b_lo > b_tol)) done = true;
            } else if (redo()) {
                guided = false;
            } else {
                // nearest samples on either side of the transition, the first
                // escaping sample
                const int before = level;
                double lo = near.lo, hi = near.hi;
                for (int pair = 0; pair < 2; ++pair) {
                    const double floor_e = pair == 0 ? -INFINITY : near.e1;
                    double v = traced && fate == RAY_ESCAPED && b > floor_e ? b : INFINITY, t = tau;
                    group_min(v, t, S);
                    keep_two(v, t, near.e1, near.te1, near.e2, near.te2);
                }
                const double e1 = near.e1 < hi ? near.e1 : hi;
                if (near.c1 >= e1) near.c1 = near.c2 = -INFINITY;   // (not below the first escaping one)
                double below = -INFINITY;   // c1 among this pass's samples
                for (int pair = 0; pair < 2; ++pair) {
                    const double roof = pair == 0 ? e1 : below;
                    double v = traced && fate != RAY_ESCAPED && b < roof ? -b : INFINITY;
                    double t = fate == RAY_CAPTURED ? tau : INFINITY;   // (no time for other ends)
                    group_min(v, t, S);
                    if (pair == 0) below = -v;
                    // the pair (c1, c2) kept by decreasing b
                    const double cb = -v;
                    if (cb > near.c1) {
                        near.c2 = near.c1;
                        near.tc2 = near.tc1;
                        near.c1 = cb;
                        near.tc1 = t;
                    } else if (cb < near.c1 && cb > near.c2) {
                        near.c2 = cb;
                        near.tc2 = t;
                    }
                }
                const double c1 = near.c1 > lo ? near.c1 : lo;
                // the levels that (c1, e1) settles: no edge strictly inside it
                while (!done) {
                    const double w = (hi - lo) / (S + 1);
                    const double q = (e1 - lo) / w;
                    int j = q >= static_cast<double>(S) ? S : static_cast<int>(q) - 1;
                    if (j < 1) j = 1;
                    while (j <= S && edge(lo, hi, w, j, S) < e1) ++j;
                    while (j > 1 && edge(lo, hi, w, j - 1, S) >= e1) --j;
                    if (!(edge(lo, hi, w, j - 1, S) <= c1)) break;
                    double nlo = lo, nhi = hi;
                    cell(nlo, nhi, w, j, S);
                    if (nlo == lo && nhi == hi) done = true;   // below the resolution of b
                    lo = nlo;
                    hi = nhi;
                    if (++level >= kMaxLevels || !(hi - lo > b_tol)) done = true;
                }
                near.lo = lo;
                near.hi = hi;
                // (a guided pass that settled nothing is followed by a uniform one)
                guided = (guide & kMay) && level >= 2 && level > before;
            }
            if (!done) start_pass();
        }
    }
    // the group's attempt total, in a fixed order
    for (int off = S / 2; off > 0; off >>= 1) used += __shfl_xor(used, off);
    if (mine && sl == 0) {
        out[2 * dir] = near.lo;
        out[2 * dir + 1] = near.hi;
        status[dir] = result;
        if (attempts) attempts[dir] = used;
    }
}

}  // namespace

hipError_t launch_boundary(const ImageConst& c, const double* dirs, int32_t n, int32_t samples,
                           double b_lo, double b_hi, double b_tol, double* out, int32_t* status,
                           int64_t* attempts, hipStream_t stream) {
    const int64_t waves = (static_cast<int64_t>(n) * samples + 63) / 64;
    const int32_t blocks = static_cast<int32_t>((waves + kBlock / 64 - 1) / (kBlock / 64));
    if (c.metric == KERR)
        hipLaunchKernelGGL(boundary_kernel<KERR>, dim3(blocks), dim3(kBlock), 0, stream, c, dirs,
                           n, samples, b_lo, b_hi, b_tol, out, status, attempts);
    else if (c.metric == EINASTO)
        hipLaunchKernelGGL(boundary_kernel<EINASTO>, dim3(blocks), dim3(kBlock), 0, stream, c,
                           dirs, n, samples, b_lo, b_hi, b_tol, out, status, attempts);
    else if (c.ex_near)
        hipLaunchKernelGGL(boundary_kernel<CNFW_NEAR>, dim3(blocks), dim3(kBlock), 0, stream, c,
                           dirs, n, samples, b_lo, b_hi, b_tol, out, status, attempts);
    else
        hipLaunchKernelGGL(boundary_kernel<CNFW>, dim3(blocks), dim3(kBlock), 0, stream, c, dirs,
                           n, samples, b_lo, b_hi, b_tol, out, status, attempts);
    return hipGetLastError();
}

}  // namespace rt
