// rt_visibility.hip -- normalised visibility amplitudes of traced images
// (Sec. 6.4): V(u,v) = sum over the pixel centres of I(X,Y) exp(-2 pi i (u X
// + v Y)) dX dY and amp(u,v) = |V(u,v)| / |V(0,0)|, the midpoint rule, at K
// arbitrary (u, v) points per image; many images in one launch.
//
// The phase factorises over the screen axes, and the pixel rows lie in pairs
// Y_c -+ a about the screen's centre row Y_c.  With S = I(Y_c - a) + I(Y_c + a)
// and D = I(Y_c - a) - I(Y_c + a) of each pair,
//   sum_y exp(-2 pi i v Y) I = exp(-2 pi i v Y_c) sum_a [cos(2 pi v a) S + i sin(2 pi v a) D],
// two real products per pixel pair where the plain sum takes four, so the work
// is two real matrix products per image (K points x folded rows x columns),
//   R_k(x) = sum_a cos(2 pi v_k a) S(a, x),   J_k(x) = sum_a sin(2 pi v_k a) D(a, x),
// done on the matrix cores in binary64 (v_mfma_f64_16x16x4, which accumulates
// with fused multiply-adds like the vector unit):
//   * a first pass sums the flux |V(0,0)|;
//   * one wavefront per work item = (image, 32 points, 64 columns, a segment
//     of the folded rows), 16 accumulator tiles; a lane reads the pixel pairs of
//     its own row and columns (a load of a wavefront is 16 columns x 4 rows) and
//     generates its own elements of the left operand, cos and sin of its point's
//     phase at its row, stepped four rows by one complex multiplication and
//     re-seeded from an exact sine and cosine every kReseed row quads (recurrence
//     error ~1e-14), in the shadow of the matrix instructions;
//   * the item's 64 columns are then summed with exp(-2 pi i (u X + v Y_c)).
// Each work item writes one partial sum per point; a last kernel adds a
// point's partials in index order, scales by dX dY and divides by the flux.
// Deterministic run to run, and the split of an image depends on its size alone.
// Points go in rounds whose partial sums fit kVisPart, one round after another.
//
// Bound by the binary64 matrix rate: a probe of independent
// v_mfma_f64_16x16x4 reaches 77 TFLOP/s on this card (71 with one wavefront
// per SIMD, so two waves suffice), where dependent-free vector FMAs hold 52
// under the same power limit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "rt_kernels.h"
#include "rt_math.h"

namespace rt {
namespace {

constexpr double kTwoPi = 6.283185307179586;
constexpr int kVisThreads = 256;            // four work items (wavefronts) per block
constexpr int kReseed = 16;                 // row quads between exact phases
constexpr int kPT = 2, kCT = 4;             // 16-point and 16-column tiles of a work item

typedef double Acc __attribute__((ext_vector_type(4)));

// Image i of a call: of the device table, or the call's only one, which comes
// with the kernel's arguments (no table to fill and copy: a single image's call
// waits for its host, and the copy was a launch of its own).
template <bool ONE>
__device__ __forceinline__ const VisImage& image_of(const VisImage* __restrict__ tab, const VisImage& one,
                                                    int i) {
    if constexpr (ONE)
        return one;
    else
        return tab[i];
}

// Flux partials, over cells of 16 columns x 4 row pairs: block b of image i takes
// every kVisFluxBlocks-th group of four cells and leaves their sum in
// fpart[i kVisFluxBlocks + b] (fixed order).
template <bool ONE>
__global__ __launch_bounds__(kVisThreads) void vis_flux_kernel(const VisImage* __restrict__ tab,
                                                               VisImage one, double* __restrict__ fpart) {
    __shared__ double sh[kVisThreads];
    const VisImage& m = image_of<ONE>(tab, one, static_cast<int>(blockIdx.y));
    const int32_t nx = m.nx, ny = m.ny, nq = m.nq;
    const int32_t h = (ny + 1) / 2;
    const int64_t cells = static_cast<int64_t>(m.nct) * nq;
    const int lane = static_cast<int>(threadIdx.x & 63), r = lane >> 4, col = lane & 15;
    double sum = 0.0;
    for (int64_t cell = 4 * static_cast<int64_t>(blockIdx.x) + (threadIdx.x >> 6); cell < cells;
         cell += 4 * kVisFluxBlocks) {
        const int32_t t = static_cast<int32_t>(cell / nq), q = static_cast<int32_t>(cell - static_cast<int64_t>(t) * nq);
        const int32_t x = 16 * t + col, y = 4 * q + r;
        double S = 0.0;
        if (x < nx && y < h) {
            const int32_t z = ny - 1 - y;
            S = m.I[static_cast<int64_t>(y) * nx + x];
            if (z > y) S += m.I[static_cast<int64_t>(z) * nx + x];   // (else the centre row of an odd screen)
        }
        sum += S;
    }
    sh[threadIdx.x] = sum;
    __syncthreads();
    for (int w = kVisThreads / 2; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) fpart[blockIdx.y * kVisFluxBlocks + blockIdx.x] = sh[0];
}

// Partial sums of V over one work item.
template <bool ONE>
__global__ __launch_bounds__(kVisThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void vis_partial_kernel(
    const VisImage* __restrict__ tab, VisImage one, int32_t n_img, int32_t n_items,
    double2* __restrict__ part) {
    const int32_t w = __builtin_amdgcn_readfirstlane(
        static_cast<int32_t>(blockIdx.x) * (kVisThreads / 64) + static_cast<int32_t>(threadIdx.x >> 6));
    if (w >= n_items) return;
    int32_t lo = 0, hi = ONE ? 0 : n_img - 1;   // the image whose items hold w
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (tab[mid].item0 <= w) lo = mid; else hi = mid - 1;
    }
    const VisImage& m = image_of<ONE>(tab, one, lo);
    // items: point groups fastest, so a block's wavefronts read the same rows
    const int32_t local = w - m.item0;
    const int32_t cell = local / m.nkg, kg = local - cell * m.nkg;
    const int32_t cb = cell / m.nseg, seg = cell - cb * m.nseg;
    const int32_t K = m.K, nq = m.nq;
    const int lane = __lane_id(), r = lane >> 4, i16 = lane & 15;
    const int32_t q0 = static_cast<int32_t>(static_cast<int64_t>(nq) * seg / m.nseg);
    const int32_t q1 = static_cast<int32_t>(static_cast<int64_t>(nq) * (seg + 1) / m.nseg);
    const int32_t k0 = kg * 16 * kPT;

    // left operand: lane (r, i16) holds point k0 + 16 p + i16 at row 4 q + r
    double tv[kPT], c[kPT], s[kPT], wc[kPT], ws[kPT];
#pragma unroll
    for (int p = 0; p < kPT; ++p) {
        const int32_t k = k0 + 16 * p + i16;
        tv[p] = k < K ? kTwoPi * m.uv[2 * k + 1] : 0.0;
        dm::sincos(tv[p] * (4.0 * m.dy), &ws[p], &wc[p]);
        c[p] = 1.0;
        s[p] = 0.0;
    }
    Acc R[kPT][kCT], J[kPT][kCT];
#pragma unroll
    for (int p = 0; p < kPT; ++p)
#pragma unroll
        for (int t = 0; t < kCT; ++t) R[p][t] = J[p][t] = Acc{0.0, 0.0, 0.0, 0.0};

    // right operand: the pair of rows y = 4 q + r and ny - 1 - y at column 64 cb +
    // 16 t + i16; rows and columns beyond the screen (clamped here) enter as zeros
    const int32_t nx = m.nx, ny = m.ny, h = (ny + 1) / 2;
    int32_t col[kCT];
    bool inside[kCT];
#pragma unroll
    for (int t = 0; t < kCT; ++t) {
        const int32_t x = 16 * (cb * kCT + t) + i16;
        inside[t] = x < nx;
        col[t] = inside[t] ? x : nx - 1;
    }
    double a[kCT], b[kCT];
    auto load = [&](int32_t q) {
        const int32_t y = 4 * q + r, yc = y < h ? y : h - 1;
        const double* top = m.I + static_cast<int64_t>(yc) * nx;
        const double* bottom = m.I + static_cast<int64_t>(ny - 1 - yc) * nx;
#pragma unroll
        for (int t = 0; t < kCT; ++t) {
            a[t] = top[col[t]];
            b[t] = bottom[col[t]];
        }
    };
    const double half = 0.5 * static_cast<double>(ny);
    load(q0);
    for (int32_t q = q0; q < q1; ++q) {
        if (((q - q0) & (kReseed - 1)) == 0) {
#pragma unroll
            for (int p = 0; p < kPT; ++p)
                dm::sincos(tv[p] * ((static_cast<double>(4 * q + r) + 0.5 - half) * m.dy), &s[p], &c[p]);
        }
        // (the centre row of an odd screen has no partner)
        const int32_t y = 4 * q + r;
        const bool row = y < h, pair = y < ny - 1 - y;
        double S[kCT], D[kCT];
#pragma unroll
        for (int t = 0; t < kCT; ++t) {
            const double s_ = pair ? a[t] + b[t] : a[t], d_ = a[t] - b[t];
            S[t] = row && inside[t] ? s_ : 0.0;
            D[t] = pair && inside[t] ? d_ : 0.0;
        }
        // the next quad's loads stay in flight under this quad's products
        load(q + 1 < q1 ? q + 1 : q);
#pragma unroll
        for (int p = 0; p < kPT; ++p)
#pragma unroll
            for (int t = 0; t < kCT; ++t) {
                R[p][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[p], S[t], R[p][t], 0, 0, 0);
                J[p][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(s[p], D[t], J[p][t], 0, 0, 0);
            }
#pragma unroll
        for (int p = 0; p < kPT; ++p) {
            const double cn = c[p] * wc[p] - s[p] * ws[p];
            s[p] = s[p] * wc[p] + c[p] * ws[p];
            c[p] = cn;
        }
    }
    // Columns.  Element v of a result tile is point r + 4 v of the point tile
    // at column i16 of the column tile.  (The phases above were taken at the
    // first row of each pair, Y_c - a, so the accumulated sine has the other
    // sign.)
    const double Yc = m.y0 + half * m.dy;
    const double X = m.x0 + (static_cast<double>(cb * 16 * kCT + i16) + 0.5) * m.dx;
    // This lane's own point, i16/2 of its row's eight, for what does not depend
    // on the column: the step to the next column tile and the phase of Y_c.  (One
    // sine and cosine of each per lane in place of eight, and sums that halve
    // what a lane carries: 57.6 -> 52 us for 1024 points of a 1024^2 image.)
    static_assert(kPT == 2, "eight points per row of lanes, two lanes each");
    const int32_t mine = k0 + 16 * (i16 >> 3) + r + 4 * (i16 >> 1 & 3);
    const double mu = mine < K ? -kTwoPi * m.uv[2 * mine] : 0.0;
    const double mv = mine < K ? -kTwoPi * m.uv[2 * mine + 1] : 0.0;
    double step_s, step_c, ys, yc;
    dm::sincos(mu * (16.0 * m.dx), &step_s, &step_c);
    dm::sincos(mv * Yc, &ys, &yc);
    double sum[8 * kPT];   // (re, im) of the row's points over this lane's columns
#pragma unroll
    for (int p = 0; p < kPT; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int j = 4 * p + v;
            const double vs = __shfl(step_s, (lane & 48) + 2 * j), vc = __shfl(step_c, (lane & 48) + 2 * j);
            const double pu = __shfl(mu, (lane & 48) + 2 * j);
            double xs, xc;
            dm::sincos(pu * X, &xs, &xc);
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int t = 0; t < kCT; ++t) {
                const double a = R[p][t][v], b = -J[p][t][v];
                re += xc * a - xs * b;
                im += xc * b + xs * a;
                const double cn = xc * vc - xs * vs;
                xs = xs * vc + xc * vs;
                xc = cn;
            }
            sum[2 * j] = re;
            sum[2 * j + 1] = im;
        }
    // Sums over the row's 16 lanes: each exchange halves the values a lane
    // carries, and lane i16 ends with value i16, of its own point.
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const bool odd = i16 >> b & 1;
#pragma unroll
        for (int j = 0; j < 8 >> b; ++j) {
            const double keep = odd ? sum[2 * j + 1] : sum[2 * j], give = odd ? sum[2 * j] : sum[2 * j + 1];
            sum[j] = keep + __shfl_xor(give, 1 << b);
        }
    }
    const double other = __shfl_xor(sum[0], 1);
    const double re = i16 & 1 ? other : sum[0], im = i16 & 1 ? sum[0] : other;
    const double out_re = re * yc - im * ys, out_im = re * ys + im * yc;
    if (mine < K)
        reinterpret_cast<double*>(part + m.part0 + static_cast<int64_t>(cell) * K + mine)[i16 & 1] =
            i16 & 1 ? out_im : out_re;
}

// V_k = dX dY sum over the work items' partials (index order), amp_k = |V_k| / |F|.
template <bool ONE>
__global__ __launch_bounds__(kVisThreads) void vis_finish_kernel(const VisImage* __restrict__ tab,
                                                                 VisImage one, const double2* __restrict__ part,
                                                                 const double* __restrict__ fpart) {
    __shared__ double sh[kVisThreads];
    static_assert(kVisFluxBlocks == kVisThreads, "one flux partial per thread");
    const VisImage& m = image_of<ONE>(tab, one, static_cast<int>(blockIdx.y));
    sh[threadIdx.x] = fpart[blockIdx.y * kVisFluxBlocks + threadIdx.x];
    __syncthreads();
    for (int w = kVisThreads / 2; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    const int32_t k = static_cast<int32_t>(blockIdx.x) * kVisThreads + threadIdx.x;
    if (k >= m.K) return;
    const double dxdy = m.dx * m.dy;
    const double f = sh[0] * dxdy;
    double re = 0.0, im = 0.0;
    const int32_t cells = m.ncb * m.nseg;
#pragma unroll 8
    for (int32_t i = 0; i < cells; ++i) {
        const double2 p = part[m.part0 + static_cast<int64_t>(i) * m.K + k];
        re += p.x;
        im += p.y;
    }
    re *= dxdy;
    im *= dxdy;
    if (m.vis) {
        m.vis[2 * k] = re;
        m.vis[2 * k + 1] = im;
    }
    if (m.amp) m.amp[k] = sqrt(re * re + im * im) / fabs(f);
}

// Points on rings: uv[j n_dirs + a] = q_j (cos phi_a, sin phi_a),
// phi_a = 2 pi a / n_angles, a < n_dirs.
__global__ void ring_points_kernel(const double* __restrict__ q, int32_t n_q, int32_t n_angles,
                                   int32_t n_dirs, double* __restrict__ uv) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= static_cast<int64_t>(n_q) * n_dirs) return;
    const int32_t j = static_cast<int32_t>(i / n_dirs);
    const int32_t a = static_cast<int32_t>(i - static_cast<int64_t>(j) * n_dirs);
    double s, c;
    dm::sincos(kTwoPi * static_cast<double>(a) / static_cast<double>(n_angles), &s, &c);
    uv[2 * i] = q[j] * c;
    uv[2 * i + 1] = q[j] * s;
}

// avg[j] = mean over the ring's n_dirs amplitudes (index order); cut[j] =
// the amplitude at phi = 0, i.e. at (u, v) = (q_j, 0).
__global__ void ring_average_kernel(const double* __restrict__ amp, int32_t n_q, int32_t n_dirs,
                                    double* __restrict__ avg, double* __restrict__ cut) {
    const int32_t j = static_cast<int32_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (j >= n_q) return;
    const double* a = amp + static_cast<int64_t>(j) * n_dirs;
    double s = 0.0;
    for (int32_t i = 0; i < n_dirs; ++i) s += a[i];
    if (avg) avg[j] = s / static_cast<double>(n_dirs);
    if (cut) cut[j] = a[0];
}

}  // namespace

// The split of an image into work items: 32 points x 64 columns x a segment of its
// rows.  An image of 1024^2 at 1024 points has 512 pairs of point and column
// blocks, which alone would leave half of the SIMDs without a wavefront: a
// segment for every 32 quads (256 image rows) or part of it.  The split is the
// image's, whatever the number of points, and with it a point's bits (1024^2, 60,000
// points: 2.47 ms with one segment, as many points allow, 2.62 with four).
void vis_layout(const VisImage* imgs, int32_t n_img, std::vector<VisImage>* entries,
                std::vector<VisRound>* rounds, int64_t* n_part) {
    entries->clear();
    rounds->assign(1, VisRound{0, 0, 0, 0});
    int64_t part = 0, most = 0;   // partial sums of the last round, of the largest
    for (int32_t i = 0; i < n_img; ++i) {
        VisImage m = imgs[i];
        m.nct = (m.nx + 15) / 16;
        m.ncb = (m.nct + kCT - 1) / kCT;
        m.nq = ((m.ny + 1) / 2 + 3) / 4;
        m.nseg = (m.nq + 31) / 32;
        const int64_t cells = static_cast<int64_t>(m.ncb) * m.nseg;
        for (int32_t left = m.K; left > 0;) {
            VisRound& r = rounds->back();
            const int64_t fit = (kVisPart - part) / cells;
            if (left <= fit)
                m.K = left;
            else if (fit >= 16 * kPT || r.n == 0)
                m.K = std::min<int32_t>(left, fit < 16 * kPT ? 16 * kPT : static_cast<int32_t>(fit / (16 * kPT)) * 16 * kPT);
            else {
                rounds->push_back(VisRound{static_cast<int32_t>(entries->size()), 0, 0, 0});
                part = 0;
                continue;
            }
            m.nkg = (m.K + 16 * kPT - 1) / (16 * kPT);
            m.item0 = static_cast<int32_t>(r.n_items);
            m.part0 = part;
            entries->push_back(m);
            ++r.n;
            r.n_items += m.nkg * cells;
            r.max_k = std::max(r.max_k, m.K);
            part += cells * m.K;
            most = std::max(most, part);
            left -= m.K;
            m.uv += 2 * static_cast<int64_t>(m.K);
            if (m.amp) m.amp += m.K;
            if (m.vis) m.vis += 2 * static_cast<int64_t>(m.K);
        }
    }
    *n_part = most;
}

template <bool ONE>
static void launch_all(const VisImage* tab, const VisImage& one, const VisRound& r, double2* part, double* fpart,
                       hipStream_t stream) {
    hipLaunchKernelGGL(vis_flux_kernel<ONE>, dim3(kVisFluxBlocks, static_cast<unsigned>(r.n)),
                       dim3(kVisThreads), 0, stream, tab, one, fpart);
    const int32_t per_block = kVisThreads / 64;
    hipLaunchKernelGGL(vis_partial_kernel<ONE>,
                       dim3(static_cast<unsigned>((r.n_items + per_block - 1) / per_block)),
                       dim3(kVisThreads), 0, stream, tab, one, r.n, static_cast<int32_t>(r.n_items), part);
    hipLaunchKernelGGL(vis_finish_kernel<ONE>,
                       dim3(static_cast<unsigned>((r.max_k + kVisThreads - 1) / kVisThreads),
                            static_cast<unsigned>(r.n)),
                       dim3(kVisThreads), 0, stream, tab, one, part, fpart);
}

hipError_t launch_visibility(const VisImage* d_entries, const VisImage* entries, const VisRound& r, double2* part,
                             double* fpart, hipStream_t stream) {
    if (r.n == 1)
        launch_all<true>(nullptr, entries[r.first], r, part, fpart, stream);
    else
        launch_all<false>(d_entries + r.first, entries[r.first], r, part, fpart, stream);
    return hipGetLastError();
}

hipError_t launch_ring_points(const double* q, int32_t n_q, int32_t n_angles, int32_t n_dirs,
                              double* uv, hipStream_t stream) {
    const int64_t n = static_cast<int64_t>(n_q) * n_dirs;
    hipLaunchKernelGGL(ring_points_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256),
                       0, stream, q, n_q, n_angles, n_dirs, uv);
    return hipGetLastError();
}

hipError_t launch_ring_average(const double* amp, int32_t n_q, int32_t n_dirs, double* avg,
                               double* cut, hipStream_t stream) {
    hipLaunchKernelGGL(ring_average_kernel, dim3(static_cast<unsigned>((n_q + 255) / 256)),
                       dim3(256), 0, stream, amp, n_q, n_dirs, avg, cut);
    return hipGetLastError();
}

}  // namespace rt
