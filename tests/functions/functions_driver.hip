// Host driver for tests/test_functions.py: the right-hand side with its
// functions taken from each policy of rt_functions.h (compiled for the host
// from the same source).
//   row = metric chi m0 m1 m2 E L R th pR pth
//   out: the six derivatives by fn::Direct, then by fn::Pinned
#include <cstdio>
#include <cstring>
#include <vector>

#include "rt_ray.h"

using namespace rt;

namespace {

template <int M>
void rhs_case(const double* a, std::vector<double>& out) {
    ImageConst c;
    std::memset(&c, 0, sizeof c);
    c.chi = a[1];
    c.chi2 = a[1] * a[1];
    if (M == EINASTO) c.inv_lam = a[2];
    if (is_cnfw(M)) {
        c.lam_c = a[2];
        c.inv_lam_c = a[3];
        c.eta_lc = a[4];
    }
    const ray::Hot k = ray::hot_of(c);
    double d[6];
    ray::rhs<M>(k, a[5], a[6], a[7], a[8], a[9], a[10], d);
    out.insert(out.end(), d, d + 6);
    ray::rhs<M>(k, a[5], a[6], a[7], a[8], a[9], a[10], d, fn::Pinned{});
    out.insert(out.end(), d, d + 6);
}

}  // namespace

int main() {
    const size_t width = 11;
    std::vector<double> in, out;
    double v;
    while (std::fread(&v, sizeof v, 1, stdin) == 1) in.push_back(v);
    if (in.size() % width) return 3;
    for (size_t i = 0; i < in.size(); i += width) {
        const double* a = &in[i];
        const int m = static_cast<int>(a[0]);
        if (m == KERR) rhs_case<KERR>(a, out);
        else if (m == EINASTO) rhs_case<EINASTO>(a, out);
        else if (m == CNFW) rhs_case<CNFW>(a, out);
        else rhs_case<CNFW_NEAR>(a, out);
    }
    std::fwrite(out.data(), sizeof(double), out.size(), stdout);
    return 0;
}
