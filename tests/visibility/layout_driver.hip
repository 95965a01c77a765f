// Host driver for tests/test_visibility_layout.py: the work split of a visibility
// call (csrc/rt_visibility.hip, linked from the same source).
//   rows of int32 (nx, ny, K); out: column blocks and row segments of each image
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "rt_kernels.h"

int main() {
    int32_t row[3];
    std::vector<int64_t> out;
    while (std::fread(row, sizeof(int32_t), 3, stdin) == 3) {
        rt::VisImage m;
        std::memset(&m, 0, sizeof m);
        m.nx = row[0];
        m.ny = row[1];
        m.K = row[2];
        int64_t n_items = 0, n_part = 0, n_fold = 0;
        rt::vis_layout(&m, 1, &n_items, &n_part, &n_fold);
        for (int64_t v : {static_cast<int64_t>(m.ncb), static_cast<int64_t>(m.nseg)}) out.push_back(v);
    }
    std::fwrite(out.data(), sizeof(int64_t), out.size(), stdout);
    return 0;
}
