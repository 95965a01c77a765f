// rt_search.h -- the shadow boundary's decisions (rt_boundary.hip): which edge a
// lane samples in a pass and how a finished pass narrows its direction's bracket.
// Host and device: `lanes` gives the S samples of a direction's pass, on the
// device one per lane of its group, on the host an array.
//
// The result is defined by multisection: level 1 divides the bracket into S + 1
// cells and keeps the one below the first escaping edge, level 2 divides that
// one, and so on until a cell is no wider than b_tol.  A pass that samples the S
// inner edges of one level gains that level (a uniform pass).  A guided pass
// samples edges two or three levels down, around a prediction of the transition,
// and gains those levels at once when it holds; the cell kept is always one whose
// two edges have been traced.
//
// The prediction: near the unstable orbit a ray's radial time tau = int dlambda
// / Sigma (which the polar motion does not enter) diverges as -a ln|b - b_c|
// with the same a on both sides.  Two escaping and two captured samples next to
// the transition give a and b_c.  The error left, in units of the bracket W
// that held the samples, is of second order, about W/2 until W ~ 1e-3 M, and
// below 1e-4 from there (measured over 12 directions of the cored-NFW and Kerr
// holes); without Sigma in the clock it stays at 2e-2.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "rt_device.h"
#include "rt_math.h"

namespace rt {
namespace search {

constexpr int kMaxLevels = 64;
constexpr int kMay = 1, kDid = 2;   // a direction may run guided passes, has run one
// The prediction lies above the transition by 0.2 W to 0.75 W of the bracket W
// (the sides' next order); taking off 0.45 W settles 4096 directions at S = 16 in
// five passes for 3294 of them and in six or seven for the others, against 2823
// without it (0.25: 3143, 0.7: 3120; the same order in four other spacetimes).
constexpr double kBias = 0.45;
// How far from rays out of order others may be, in units of the extent of those that
// have been seen (redo).
constexpr double kFar = 16.0;

// What a direction keeps between passes: its two nearest escaping samples with
// their radial times (b_c < e1 < e2; infinity where there is none), its two
// nearest captured ones (c2 < c1 < b_c; minus infinity), its bracket, the last one
// that uniform passes alone had reached, with its level, and the range of a check.
struct Nearest {
    double e1, te1, e2, te2, c1, tc1, c2, tc2;
    double lo, hi, ulo, uhi, from, to;
    int ulevel;
};

// How far a direction is (alike in all its lanes).
struct Course {
    int level;     // levels of the multisection done (-1: bracket unchecked)
    int guide;     // kMay, kDid
    bool guided;   // the next pass is a guided one
    int check;     // edges of the bracket checked (-1: no check under way)
    bool done;
};

// One lane's part in a pass: its sample b and, once its ray has ended, the fate
// and the radial time.
struct Sample {
    double b, tau;
    bool traced;
    int32_t fate;
};

// The search's constants.
struct Search {
    int S;
    double b_lo, b_hi, b_tol;
    // Guided passes stop at cells of this width: below it rounding may decide
    // single rays' fates, and the levels left go edge by edge from the first.
    __host__ __device__ __forceinline__ double finest() const { return fmax(b_tol, 1e-11 * b_hi); }
};

// Edge j of cell division (lo, hi, w), j = 0..S + 1 (no contraction: every use
// gives the same bits).
__host__ __device__ __forceinline__ double edge(double lo, double hi, double w, int j, int S) {
    if (j <= 0) return lo;
    if (j > S) return hi;
    const double t = static_cast<double>(j) * w;
    return lo + t;
}

// The first edge j = 1..S + 1 that is not below e (e above lo, at most hi).
__host__ __device__ __forceinline__ int first_edge(double lo, double hi, double w, double e, int S) {
    const double r = (e - lo) / w;
    int j = r >= static_cast<double>(S) ? S : static_cast<int>(r) - 1;
    if (j < 1) j = 1;
    while (j <= S && edge(lo, hi, w, j, S) < e) ++j;
    while (j > 1 && edge(lo, hi, w, j - 1, S) >= e) --j;
    return j;
}

// Cell j = 1..S + 1 of (lo, hi, w).
__host__ __device__ __forceinline__ void cell(double& lo, double& hi, double w, int j, int S) {
    const double nlo = edge(lo, hi, w, j - 1, S), nhi = edge(lo, hi, w, j, S);
    lo = nlo;
    hi = nhi;
}

__host__ __device__ __forceinline__ float log2_quotient(double a, double b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_logf(static_cast<float>(a * dm::recip1(b)));
#else
    return std::log2(static_cast<float>(a / b));
#endif
}

// The transition predicted from n: x in (c1, e1) where the two sides' logarithmic
// slopes agree, by bisection.  False without four finite samples that diverge
// towards the transition.
template <class N>
__host__ __device__ __forceinline__ bool predict(const N& n, double* x_out) {
    const double c1 = n.c1, c2 = n.c2, e1 = n.e1, e2 = n.e2;
    const double De = n.te1 - n.te2, Dc = n.tc1 - n.tc2;
    if (!(c2 > -INFINITY && e2 < INFINITY && De > 0.0 && Dc > 0.0 && De < INFINITY && Dc < INFINITY))
        return false;
    double a = c1, b = e1;
    for (int it = 0; it < 32; ++it) {
        const double x = 0.5 * (a + b);
        const float fe = log2_quotient(e2 - x, e1 - x), fc = log2_quotient(x - c2, x - c1);
        if (De * fc > Dc * fe) a = x; else b = x;
    }
    *x_out = 0.5 * (a + b);
    return true;
}

// The bracket after a uniform pass, from its first escaping edge (S + 1: none).
// Returns whether the search has ended.
__host__ __device__ __forceinline__ bool narrow_uniform(const Search& q, int first, double& lo, double& hi, int& level) {
    const double was_lo = lo, was_hi = hi;
    cell(lo, hi, (hi - lo) / (q.S + 1), first, q.S);
    return ++level >= kMaxLevels || (lo == was_lo && hi == was_hi) || !(hi - lo > q.b_tol);
}

template <class N>
__host__ __device__ __forceinline__ void begin(const Search& q, N& n, Course& s) {
    n.e1 = n.e2 = INFINITY;
    n.c1 = n.c2 = -INFINITY;
    n.te1 = n.te2 = n.tc1 = n.tc2 = 0.0;
    n.lo = n.ulo = q.b_lo;
    n.hi = n.uhi = q.b_hi;
    n.ulevel = 0;
    s.level = -1;
    s.guide = kMay;
    s.guided = false;
    s.check = -1;
    s.done = false;
}

// Sample `at` of the check of (n.lo, n.hi): the edges that decide the levels from
// (n.ulo, n.uhi) down to it, of each up to the first that is to escape, within
// n.from..n.to.  Below the bracket's upper end they end inside and from there they
// escape, if it is multisection's.  Not traced past the last of them.
template <class N>
__host__ __device__ __forceinline__ Sample check_edge(const Search& q, int at, const N& n, const Course& s) {
    const double hi = n.hi, from = n.from, to = n.to;
    double l = n.ulo, h = n.uhi;
    const int levels = s.level - n.ulevel;
    for (int m = 0; m < levels; ++m) {
        const double w = (h - l) / (q.S + 1);
        const int j = first_edge(l, h, w, hi, q.S), first = from > l ? first_edge(l, h, w, from, q.S) : 1;
        int last = j < q.S ? j : q.S;
        if (last >= first && !(edge(l, h, w, last, q.S) <= to)) --last;   // (the others are below the bracket)
        if (first + at <= last) return Sample{edge(l, h, w, first + at, q.S), 0.0, true, 0};
        if (last >= first) at -= last - first + 1;
        cell(l, h, w, j, q.S);
    }
    return Sample{0.0, 0.0, false, 0};
}

// Lane sl's sample of the next pass along a direction of this length (b times it is
// the impact parameter in M).  Level -1 checks the bracket: sample 0 at
// b_lo must stay inside, sample 1 at b_hi must escape.
template <class N>
__host__ __device__ __forceinline__ Sample choose(const Search& q, double length, int sl, const N& n,
                                                   Course& s) {
    const int S = q.S;
    const double lo = n.lo, hi = n.hi;
    const double w = (hi - lo) / (S + 1);
    Sample p{0.0, 0.0, true, 0};
    if (s.level < 0) {
        p.b = sl == 0 ? q.b_lo : q.b_hi;
        p.traced = sl < 2;
        return p;
    }
    if (s.check >= 0) return check_edge(q, s.check + sl, n, s);
    // The finest level, at most three down, whose cells the prediction
    // is expected to miss by no more than S / 4.
    const double W = (hi - lo) * length;
    const double miss = 0.5 * W + 3e-4;   // in units of the bracket
    int m = 1;
    double cells = miss * (S + 1);
    while (m < 3 && cells * (S + 1) <= 0.25 * S) {
        ++m;
        cells *= S + 1;
    }
    double x = 0.0;
    if (s.guided && m > 1 && w > q.finest() && predict(n, &x)) {
        s.guide |= kDid;
        // The S - S/4 edges of that level (or of the last before b_tol)
        // nearest to the prediction, and S/4 of the level above in
        // case it misses by more.
        x = fmax(x - kBias * W * (hi - lo), lo);
        const int coarse = S / 4;
        const bool fine = sl >= coarse;
        const int target = fine ? m : m - 1;
        double l = lo, h = hi, lw = w;
        int j = 0, at = 1;
        for (;; ++at) {
            lw = (h - l) / (S + 1);
            const double r = (x - l) / lw;
            j = r >= static_cast<double>(S) ? S + 1 : static_cast<int>(r) + 1;
            if (j < 1) j = 1;
            if (at >= target) break;
            double nl = l, nh = h;
            cell(nl, nh, lw, j, S);
            if (!(nh - nl > q.finest())) break;   // the last level
            l = nl;
            h = nh;
        }
        const int idx = fine ? j - (S - coarse) / 2 + (sl - coarse) : j - coarse / 2 + sl;
        p.traced = idx >= 1 && idx <= S && (fine || at == target);
        p.b = edge(l, h, lw, idx, S);
    } else {
        p.b = edge(lo, hi, w, sl + 1, S);
    }
    return p;
}

// Takes sample (v, t) into the ordered pair (a, ta), (b, tb), a < b.
template <class D>
__host__ __device__ __forceinline__ void keep_two(double v, double t, D& a, D& ta, D& b, D& tb) {
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

// Back to the last bracket that uniform passes had reached.
template <class N>
__host__ __device__ __forceinline__ void restart(N& n, Course& s) {
    n.lo = n.ulo;
    n.hi = n.uhi;
    s.level = n.ulevel;
}

// Whether a finished pass's samples are dropped.  The edges that guided passes
// leave out do not matter as long as fates are in order, captured below the
// transition and escaping above.  A sample that ended inside above one that
// escaped is out of order (below `finest` passes are uniform in any case): the
// direction goes on by uniform passes from the bracket that it had, if those of
// the edges left out that lie within kFar times the extent of what is out of order
// turn out as the bracket supposes.  Else, or after a ray that ran out of attempts
// or whose error estimate was not finite (it counts as inside wherever it is), from
// the last bracket that uniform passes had reached.
//   200 calls of 4096 directions (cored NFW): mean 16.7 ms and largest 28 without
// the check, 16.9 and 32 with it, 17.2 and 40 with 256 extents, 18.2 and 47 from the
// uniform bracket always; the same brackets.  On scripted rays whose transition jumps
// hundreds of times within the jumps' size, 208, 52, 20 and none of 89,875 such
// directions ended beside multisection's bracket; where the jumps are farther
// apart, none.
template <class Lanes, class N>
__host__ __device__ __forceinline__ bool redo(const Search& q, const Lanes& lanes, N& n, Course& s) {
    double out_b, in_b, unused;
    lanes.least([](const Sample& p, double* u) {
        *u = 0.0;
        return p.traced && p.fate == RAY_ESCAPED ? p.b : INFINITY;
    }, &out_b, &unused);
    lanes.least([](const Sample& p, double* u) {
        *u = 0.0;
        return p.traced && p.fate != RAY_ESCAPED ? -p.b : INFINITY;
    }, &in_b, &unused);
    out_b = fmin(out_b, n.e1);
    in_b = fmax(-in_b, n.c1);
    const bool lost = lanes.any([](const Sample& p) {
        return p.fate != 0 && p.fate != RAY_ESCAPED && p.fate != RAY_CAPTURED;
    });
    const bool order = in_b > out_b && n.hi - n.lo > q.finest();
    if (!(lost || order) || !(s.guide & kMay)) return false;
    const bool drop = s.guide & kDid;
    s.guide = 0;
    if (drop) {
        const double far = kFar * (in_b - out_b);
        n.from = out_b - far;
        n.to = in_b + far;
        if (lost) restart(n, s); else s.check = 0;
        n.e1 = n.e2 = INFINITY;
        n.c1 = n.c2 = -INFINITY;
    }
    return drop;
}

// Narrows the bracket by a finished pass of level >= 0 (or has the next pass
// search from where redo put it).
template <class Lanes, class N>
__host__ __device__ __forceinline__ void narrow(const Search& q, const Lanes& lanes, N& n, Course& s) {
    const int S = q.S;
    if (s.check >= 0) {
        const double hi = n.hi;
        const bool other = lanes.any([&](const Sample& p) { return p.traced && (p.fate == RAY_ESCAPED) != (p.b >= hi); });
        if (other) restart(n, s);
        s.check = other || lanes.any([](const Sample& p) { return !p.traced; }) ? -1 : s.check + S;
        return;
    }
    if (redo(q, lanes, n, s)) {
        s.guided = false;
        return;
    }
    // nearest samples on either side of the transition, the first
    // escaping sample
    const int before = s.level;
    double lo = n.lo, hi = n.hi;
    for (int pair = 0; pair < 2; ++pair) {
        const double floor_e = pair == 0 ? -INFINITY : n.e1;
        double v, t;
        lanes.least([&](const Sample& p, double* u) {
            *u = p.tau;
            return p.traced && p.fate == RAY_ESCAPED && p.b > floor_e ? p.b : INFINITY;
        }, &v, &t);
        keep_two(v, t, n.e1, n.te1, n.e2, n.te2);
    }
    const double e1 = n.e1 < hi ? n.e1 : hi;
    if (n.c1 >= e1) n.c1 = n.c2 = -INFINITY;   // (not below the first escaping one)
    double below = -INFINITY;   // c1 among this pass's samples
    for (int pair = 0; pair < 2; ++pair) {
        const double roof = pair == 0 ? e1 : below;
        double v, t;
        lanes.least([&](const Sample& p, double* u) {
            *u = p.fate == RAY_CAPTURED ? p.tau : INFINITY;   // (no time for other ends)
            return p.traced && p.fate != RAY_ESCAPED && p.b < roof ? -p.b : INFINITY;
        }, &v, &t);
        if (pair == 0) below = -v;
        // the pair (c1, c2) kept by decreasing b
        const double cb = -v;
        if (cb > n.c1) {
            n.c2 = n.c1;
            n.tc2 = n.tc1;
            n.c1 = cb;
            n.tc1 = t;
        } else if (cb < n.c1 && cb > n.c2) {
            n.c2 = cb;
            n.tc2 = t;
        }
    }
    const double c1 = n.c1 > lo ? n.c1 : lo;
    // the levels that (c1, e1) settles: no edge strictly inside it
    while (!s.done) {
        const double w = (hi - lo) / (S + 1);
        const int j = first_edge(lo, hi, w, e1, S);
        if (!(edge(lo, hi, w, j - 1, S) <= c1)) break;
        double nlo = lo, nhi = hi;
        cell(nlo, nhi, w, j, S);
        if (nlo == lo && nhi == hi) s.done = true;   // below the resolution of b
        lo = nlo;
        hi = nhi;
        if (++s.level >= kMaxLevels || !(hi - lo > q.b_tol)) s.done = true;
    }
    n.lo = lo;
    n.hi = hi;
    if (!(s.guide & kDid)) {
        n.ulo = lo;
        n.uhi = hi;
        n.ulevel = s.level;
    }
    // (a guided pass that settled nothing is followed by a uniform one)
    s.guided = (s.guide & kMay) && s.level >= 2 && s.level > before;
}

}  // namespace search
}  // namespace rt
