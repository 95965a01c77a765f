// Host driver for tests/test_claims.py: the trace kernels' claims of tile parts
// (paper_2605_05635_amd/csrc/rt_ray.h, compiled for the host from the same source).
//   rows of int64 (nx, ny, tile_w, tile_h, fine_from, wavefronts, seed)
// For each, `wavefronts` claimers take turns in a pseudo-random order until the
// queue is dry; out: how often each pixel was handed out, nx * ny values.
#include <cstdint>
#include <cstdio>
#include <numeric>
#include <vector>

#include "rt_ray.h"

int main() {
    int64_t row[7];
    std::vector<int64_t> out;
    while (std::fread(row, sizeof(int64_t), 7, stdin) == 7) {
        const int32_t nx = static_cast<int32_t>(row[0]), ny = static_cast<int32_t>(row[1]);
        rt::LaunchShape shape{64, static_cast<int32_t>(row[2]), static_cast<int32_t>(row[3])};
        std::vector<int32_t> order(static_cast<size_t>((nx + shape.tile_w - 1) / shape.tile_w) *
                                   ((ny + shape.tile_h - 1) / shape.tile_h));
        std::iota(order.rbegin(), order.rend(), 0);
        shape.order = order.data();
        shape.fine_from = row[4];
        std::vector<int64_t> seen(static_cast<size_t>(nx) * ny, 0);
        std::vector<rt::ray::TileClaim> wave(static_cast<size_t>(row[5]), rt::ray::TileClaim{0, 0, 1, 1.0f, 0, 0});
        uint64_t rng = static_cast<uint64_t>(row[6]), queue = 0;
        size_t live = wave.size();
        while (live > 0) {
            rng = rng * 6364136223846793005ull + 1442695040888963407ull;
            const size_t i = static_cast<size_t>(rng >> 33) % live;
            rt::ray::TileClaim& t = wave[i];
            int64_t next = 0, end = 0;
            auto add = [&](int n) {
                const uint64_t q = queue;
                queue += static_cast<uint64_t>(n);
                return static_cast<int64_t>(q);
            };
            if (!rt::ray::claim_parts(shape, nx, ny, t, next, end, add))
                std::swap(wave[i], wave[--live]);
            else
                for (int64_t p = next; p < end; ++p) {
                    const rt::ray::Pixel px = rt::ray::claimed(shape, nx, ny, t, p);
                    if (px.ix < 0 || px.ix >= nx || px.iy < 0 || px.iy >= ny) return 4;
                    ++seen[static_cast<size_t>(px.pix)];
                }
        }
        out.insert(out.end(), seen.begin(), seen.end());
    }
    std::fwrite(out.data(), sizeof(int64_t), out.size(), stdout);
    return 0;
}
