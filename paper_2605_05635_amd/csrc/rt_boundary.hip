// rt_boundary.hip -- gfx950 kernel of the shadow-boundary search (Sec. 4.1,
// eqs. (78)-(79)): along a screen direction (cos psi, sin psi), the impact
// parameter b at which the rays from X = b cos psi, Y = b sin psi turn from
// captured to escaping.  A wavefront holds 64 / S directions, S lanes each
// (S = 64, 32 or 16 samples per pass), and a pass traces one ray per lane.
//
// rt_search.h says which edges a pass samples and what it settles: the bracket is
// multisection's, level by level.  Every ray of a late pass winds around the photon
// shell, so passes are what costs: nine uniform ones at S = 16 from 7 M to 1e-10 M, the
// last of rays of up to 1716 attempts near the polar axis, one after another; guided
// ones settle two or three levels at once.
//
// Directions advance independently, each from pass to pass as soon as its own
// rays end.  4096 directions at S = 16, cored NFW chi = 0.94: 21.7 ms by uniform
// passes, 14.7 by guided ones (five to seven passes in place of nine); 500 at S = 64:
// 14.0 and 9.7 ms.
// What is left is the longest direction's chain, 5924 attempts of 2.4 us; 21 to 32
// ms in one call of ten, where some direction came out of order (search::redo).
#include "rt_ray.h"
#include "rt_search.h"

namespace rt {
namespace {

using namespace ray;

// Looser integrations search by uniform passes.  Fates are out of order within the
// integration's error of the transition, where an accept or reject decision flips
// between neighbouring rays, and samples that a guided pass leaves out can
// then miss a flip: with guided passes at every tolerance the bracket was another
// one for none of 184,320 directions at 1e-8 (S = 16) and of 98,304 at 1e-7, for 17 of
// 86,016 at 1e-6 and for 71 of 19,400 from 1e-5 to 1e-2 (one in 17 from 1e-6 to
// 1e-2 without the test of order in search::redo).
constexpr double kGuidedTol = 1e-7;

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

// The samples of a group's pass, one per lane.
struct GroupLanes {
    const search::Sample& mine;
    int S;
    template <class F>
    __device__ __forceinline__ void least(F f, double* v, double* t) const {
        *v = f(mine, t);
        group_min(*v, *t, S);
    }
    template <class F>
    __device__ __forceinline__ int any(F f) const {
        int m = f(mine);
        for (int off = 1; off < S; off <<= 1) m |= __shfl_xor(m, off);
        return m;
    }
};

// GUIDED passes where they may run, else uniform ones, which need neither the
// radial time nor the nearest samples (with both kinds in one kernel, uniform
// searches took 3 to 6 % longer: Kerr at a tolerance of 1e-5 5.64 -> 5.37 ms).  Registers as the trace kernel's, the
// tableau not pinned; the guided kernels of Einasto and of the near cored NFW
// spill 30 and 33 of them, in the code between passes.
template <int METRIC, bool GUIDED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void boundary_kernel(
    ImageConst c, const double* __restrict__ dirs, int32_t n, int32_t S, double b_lo, double b_hi,
    double b_tol, double* __restrict__ out, int32_t* __restrict__ status,
    int64_t* __restrict__ attempts) {
    __shared__ search::Nearest kept[GUIDED ? kBlock / 16 : 1];   // one per direction, written alike by all its lanes
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
    const search::Search q{S, b_lo, b_hi, b_tol};
    volatile search::Nearest& near = kept[GUIDED ? (threadIdx.x / 64) * 4 + grp : 0];
    search::Course course{};
    double lo = b_lo, hi = b_hi;   // the bracket of uniform passes
    course.level = -1;
    if constexpr (GUIDED) search::begin(q, near, course);
    course.done = !mine;
    int64_t used = 0;        // this lane's step attempts
    int32_t result = 1;      // bracket without the transition, until checked
    // Each group runs its passes on its own: when the last of its rays ends it
    // narrows its bracket and starts its next pass at once, while the other
    // groups' rays are still in flight.
    Ray r;
    search::Sample p{0.0, 0.0, false, 0};   // this lane's sample
    bool active = false;                    // its ray is in flight
    auto start_pass = [&]() {
        const double ux = dirs[2 * dir], uy = dirs[2 * dir + 1];
        if constexpr (GUIDED) {
            p = search::choose(q, sqrt(ux * ux + uy * uy), sl, near, course);
        } else {
            p.b = course.level < 0 ? (sl == 0 ? b_lo : b_hi) : search::edge(lo, hi, (hi - lo) / (S + 1), sl + 1, S);
            p.traced = course.level >= 0 || sl < 2;
            p.fate = 0;
        }
        active = p.traced;
        if (active) start_ray_dir<METRIC>(c, k, screen_dir_xy(c, p.b * ux, p.b * uy), 0, r, fns);
    };
    if (!course.done) start_pass();
    while (__ballot(!course.done) != 0ull) {
        if (active) {
            const int32_t st = attempt<METRIC, StageNone, false, fn::Pinned, true>(k, none, 0, r, StageNone{}, fns);
            if (st != 0) {
                active = false;
                p.fate = st;
                // the radial time at the stop radius itself
                const double stop = st == RAY_ESCAPED ? k.r_esc : k.r_stop;
                if constexpr (GUIDED) p.tau = r.tau + (stop - r.y[1]) * (r.iS / r.k1[1]);
                used += r.attempts;
            }
        }
        const unsigned long long busy = (__ballot(active) >> (grp * S)) & gmask;
        const unsigned long long esc = (__ballot(p.fate == RAY_ESCAPED) >> (grp * S)) & gmask;
        if (!course.done && busy == 0ull) {
            // the group's pass is complete
            if (course.level < 0) {
                if ((esc & 1ull) || !(esc & 2ull)) {
                    course.done = true;
                } else {
                    result = 0;
                }
                course.level = 0;
                if (!(b_hi - b_lo > b_tol)) course.done = true;
            } else if constexpr (GUIDED) {
                search::narrow(q, GroupLanes{p, S}, near, course);
            } else {
                course.done = search::narrow_uniform(q, esc != 0ull ? __ffsll(static_cast<long long>(esc)) : S + 1,
                                                     lo, hi, course.level);
            }
            if (!course.done) start_pass();
        }
    }
    // the group's attempt total, in a fixed order
    for (int off = S / 2; off > 0; off >>= 1) used += __shfl_xor(used, off);
    if (mine && sl == 0) {
        out[2 * dir] = GUIDED ? near.lo : lo;
        out[2 * dir + 1] = GUIDED ? near.hi : hi;
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
    // (a caller that counts attempts gets the count of uniform passes)
    const bool guided = attempts == nullptr && std::fmax(c.rtol, c.atol) <= kGuidedTol;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, stream, c, dirs, n, samples, b_lo, b_hi,
                           b_tol, out, status, attempts);
    };
    if (c.metric == KERR)
        guided ? launch(boundary_kernel<KERR, true>) : launch(boundary_kernel<KERR, false>);
    else if (c.metric == EINASTO)
        guided ? launch(boundary_kernel<EINASTO, true>) : launch(boundary_kernel<EINASTO, false>);
    else if (c.ex_near)
        guided ? launch(boundary_kernel<CNFW_NEAR, true>) : launch(boundary_kernel<CNFW_NEAR, false>);
    else
        guided ? launch(boundary_kernel<CNFW, true>) : launch(boundary_kernel<CNFW, false>);
    return hipGetLastError();
}

}  // namespace rt
