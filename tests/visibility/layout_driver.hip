// Host driver for tests/test_visibility_layout.py: the work split of a visibility
// call (csrc/rt_visibility.hip, linked from the same source).
//   rows of int32 (nx, ny, K, copies); out: column blocks and row segments of each image,
//   the call's partial sums, its rounds, the points that its entries take of copy 0 in
//   order without a gap or an overlap, and of all copies
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "rt_kernels.h"

int main() {
    int32_t row[4];
    std::vector<int64_t> out;
    while (std::fread(row, sizeof(int32_t), 4, stdin) == 4) {
        rt::VisImage m;
        std::memset(&m, 0, sizeof m);
        m.nx = row[0];
        m.ny = row[1];
        m.K = row[2];
        std::vector<double> uv(static_cast<size_t>(2) * m.K);
        std::vector<rt::VisImage> images, entries;
        for (int i = 0; i < row[3]; ++i) {
            m.uv = uv.data();
            m.I = uv.data() + i;   // (to tell the copies apart)
            images.push_back(m);
        }
        std::vector<rt::VisRound> rounds;
        int64_t n_part = 0, in_order = 0, all = 0;
        rt::vis_layout(images.data(), row[3], &entries, &rounds, &n_part);
        for (const rt::VisRound& r : rounds) {
            int64_t part = 0, items = 0;
            for (int32_t i = r.first; i < r.first + r.n; ++i) {
                const rt::VisImage& e = entries[static_cast<size_t>(i)];
                const int64_t cells = static_cast<int64_t>(e.ncb) * e.nseg;
                if (e.part0 != part || e.item0 != items || e.nkg != (e.K + 31) / 32 || e.K > r.max_k) return 4;
                part += cells * e.K;
                items += cells * e.nkg;
                if (e.I == uv.data() && e.uv == uv.data() + 2 * in_order) in_order += e.K;
                all += e.K;
            }
            if (part > n_part || items != r.n_items || items >= (int64_t(1) << 31)) return 5;
        }
        for (int64_t v : {static_cast<int64_t>(entries[0].ncb), static_cast<int64_t>(entries[0].nseg), n_part,
                          static_cast<int64_t>(rounds.size()), in_order, all})
            out.push_back(v);
    }
    std::fwrite(out.data(), sizeof(int64_t), out.size(), stdout);
    return 0;
}
