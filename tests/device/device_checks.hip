// Device checks for tests/test_gpu_device_functions.py and tests/test_gpu_scan_bits.py:
// kernels that evaluate the headers' functions on given arguments (device pointers;
// built beside the library).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "rt.h"
#include "rt_ray.h"
#include "rt_scan.h"

using namespace rt;

namespace {

__global__ void sqrt_kernel(const double* __restrict__ x, double* __restrict__ fast, double* __restrict__ ieee, int32_t n) {
    const int32_t i = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= n) return;
    fast[i] = dm::sqrt_normal(x[i]);
    ieee[i] = sqrt(x[i]);
}

// Ten values of one policy at (R, theta, x, u): the functions of the right-hand side
// and of the thick disc's source.
constexpr int kValues = 10;
template <int METRIC, class T>
__device__ void values(const T& tb, const ray::Hot& k, const double* a, double* out) {
    double s, c, F, dF, d[6];
    fn::signed_sincos(tb, a[1], &s, &c);
    fn::mass_function<METRIC>(tb, k, a[0], F, dF);
    ray::rhs<METRIC>(k, 1.01, 3.7, a[0], a[1], -0.8, 2.1, d, tb);
    const double v[kValues] = {s, c, F, dF, fn::exp(tb, a[2]), fn::log1p(tb, a[3]), d[0], d[3], d[4], d[5]};
    for (int j = 0; j < kValues; ++j) out[j] = v[j];
}

// out [n][3][kValues]: fn::Direct, fn::Pinned, fn::PinnedThick
template <int METRIC>
__global__ void policies_kernel(ImageConst c, const double* __restrict__ rows, double* __restrict__ out, int32_t n) {
    const int32_t i = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= n) return;
    const ray::Hot k = ray::hot_of(c);
    double* o = out + static_cast<int64_t>(i) * 3 * kValues;
    values<METRIC>(fn::Direct{}, k, rows + 4 * i, o);
    values<METRIC>(fn::pin<METRIC>(), k, rows + 4 * i, o + kValues);
    values<METRIC>(fn::pin<METRIC, true>(), k, rows + 4 * i, o + 2 * kValues);
}

// The serial searches of rt_scan.h, one point per lane.
__global__ __launch_bounds__(64) void serial_scan_kernel(const rt_scan_point* __restrict__ pts, double* __restrict__ out,
                                                         int32_t n) {
    const int32_t i = static_cast<int32_t>(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= n) return;
    const rt_scan_point q = pts[i];
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
    const double nan = __builtin_nan("");
    double res[4] = {nan, nan, nan, nan}, r, chi_e, r_e;
    if (scan::largest_root(c, c.chi2, &r)) res[0] = r;
    if (scan::largest_root(c, c.chi2 * co * co, &r)) res[1] = r;
    if (scan::extremal_spin(c, &chi_e, &r_e)) {
        res[2] = chi_e;
        res[3] = r_e;
    }
    for (int j = 0; j < 4; ++j) out[4 * i + j] = res[j];
}

}  // namespace

extern "C" {

int check_sqrt(const double* x, double* fast, double* ieee, int32_t n) {
    hipLaunchKernelGGL(sqrt_kernel, dim3((n + 255) / 256), dim3(256), 0, nullptr, x, fast, ieee, n);
    return hipGetLastError();
}

// m: the metric's constants (1/lambda_E; lambda_c, 1/lambda_c, eta lambda_c)
int check_policies(int32_t metric, double chi, const double* m, const double* rows, double* out, int32_t n) {
    ImageConst c{};
    c.chi = chi;
    c.chi2 = chi * chi;
    if (metric == EINASTO) c.inv_lam = m[0];
    if (is_cnfw(metric)) {
        c.lam_c = m[0];
        c.inv_lam_c = m[1];
        c.eta_lc = m[2];
    }
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((n + 255) / 256), dim3(256), 0, nullptr, c, rows, out, n);
    };
    if (metric == KERR) launch(policies_kernel<KERR>);
    else if (metric == EINASTO) launch(policies_kernel<EINASTO>);
    else if (metric == CNFW) launch(policies_kernel<CNFW>);
    else launch(policies_kernel<CNFW_NEAR>);
    return hipGetLastError();
}

int serial_scan(const rt_scan_point* pts, double* out, int32_t n) {
    hipLaunchKernelGGL(serial_scan_kernel, dim3((n + 63) / 64), dim3(64), 0, nullptr, pts, out, n);
    return hipGetLastError();
}

}  // extern "C"
