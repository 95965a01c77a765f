// Host driver for tests/test_search.py: the shadow boundary's decisions
// (paper_2605_05635_amd/csrc/rt_search.h, compiled for the host from the same source) on scripted rays.
//   row = S b_lo b_hi b_tol b_c jump period lost seed length
// A ray at b escapes above b_c + shift(b), a step function of b as an accept or reject decision that flips
// between neighbouring rays makes it: on each interval of length `period` another value within +-jump.  Within
// `lost` of b_c it runs out of attempts with probability 1/4.  `length` is the direction's.
//   out: lo, hi, passes, the samples traced, whether a pass was dropped, the range that was checked then
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "rt_search.h"

namespace {

using namespace rt;

double hashed(double x, uint64_t seed) {
    uint64_t z;
    std::memcpy(&z, &x, sizeof z);
    z += seed * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return static_cast<double>((z ^ (z >> 31)) >> 11) * 0x1p-53;
}

struct ArrayLanes {
    const std::vector<search::Sample>& all;
    template <class F>
    void least(F f, double* v, double* t) const {
        *v = f(all[0], t);
        for (const search::Sample& p : all) {
            double u;
            const double x = f(p, &u);
            if (x < *v) {
                *v = x;
                *t = u;
            }
        }
    }
    template <class F>
    int any(F f) const {
        int m = 0;
        for (const search::Sample& p : all) m |= f(p);
        return m;
    }
};

void ray(const double* a, search::Sample& p) {
    const double b_c = a[4], d = p.b - b_c;
    const uint64_t seed = static_cast<uint64_t>(a[8]);
    const double shift = a[5] * (2.0 * hashed(std::floor(d / a[6]), seed) - 1.0);
    const bool escapes = d > shift;
    p.fate = escapes ? RAY_ESCAPED : RAY_CAPTURED;
    if (std::fabs(d) < a[7] && hashed(p.b, seed + 1) < 0.25) p.fate = RAY_STEP_LIMIT;
    p.tau = 40.0 - 6.0 * std::log(std::fabs(d) / b_c + 1e-300) + (escapes ? 2.0 : -1.5) * (d / b_c);
}

}  // namespace

int main() {
    double a[10];
    std::vector<double> out;
    while (std::fread(a, sizeof(double), 10, stdin) == 10) {
        const search::Search q{static_cast<int>(a[0]), a[1], a[2], a[3]};
        search::Nearest near;
        search::Course course;
        search::begin(q, near, course);
        std::vector<search::Sample> lanes(static_cast<size_t>(q.S));
        double passes = 0.0, traced = 0.0, dropped = 0.0, from = -INFINITY, to = INFINITY;
        course.level = 0;
        while (!course.done) {
            for (int sl = 0; sl < q.S; ++sl) {
                lanes[sl] = search::choose(q, a[9], sl, near, course);
                if (lanes[sl].traced) {
                    ray(a, lanes[sl]);
                    traced += 1.0;
                }
            }
            passes += 1.0;
            const bool did = course.guide & search::kDid;
            search::narrow(q, ArrayLanes{lanes}, near, course);
            if (did && course.guide == 0) dropped = 1.0;
            if (course.check >= 0) {
                from = near.from;
                to = near.to;
            }
        }
        for (double v : {near.lo, near.hi, passes, traced, dropped, from, to}) out.push_back(v);
    }
    std::fwrite(out.data(), sizeof(double), out.size(), stdout);
    return 0;
}
