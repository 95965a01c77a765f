"""The work split of the visibility sums (rt_visibility.hip, built for the host).  It
depends on the image alone, so a point's sum is the same bits however many other
points a call asks for; and the scratch of a call, its partial sums, is no more
than four for each point and block of 64 columns where the screen has no more than
1024 rows, and bounded for any."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_05635_amd", "csrc")
SIZES = [(1, 1), (16, 16), (17, 300), (64, 255), (64, 256), (64, 257), (65, 1000), (128, 1024), (301, 187), (333, 777),
         (512, 512), (1024, 1024), (4096, 4096), (24, 8192), (8192, 24), (1 << 20, 3), (3, 1 << 20)]
POINTS = [1, 31, 32, 33, 64, 1024, 2000, 2048, 4097, 60000, 1 << 22]
BOUND = 1 << 24   # partial sums of a round (256 MB)


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("visibility") / "layout_driver")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=on",
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "visibility", "layout_driver.hip"),
                    os.path.join(CSRC, "rt_visibility.hip"), "-o", exe], check=True, capture_output=True)

    def run(rows):
        out = subprocess.run([exe], input=np.array(rows, dtype=np.int32).tobytes(), capture_output=True, check=True)
        return np.frombuffer(out.stdout, dtype=np.int64).reshape(len(rows), 6)
    return run


def test_split_of_an_image(layout):
    out = layout([(nx, ny, K, 1) for nx, ny in SIZES for K in POINTS])
    per = out[:, :2].reshape(len(SIZES), len(POINTS), 2)
    assert (per == per[:, :1]).all()


@pytest.mark.parametrize("copies", [1, 3, 64])
def test_scratch_and_rounds(layout, copies):
    rows = [(nx, ny, K, copies) for nx, ny in SIZES for K in POINTS]
    for (nx, ny, K, n), (ncb, nseg, part, rounds, in_order, every) in zip(rows, layout(rows)):
        assert in_order == K and every == n * K
        if ny <= 1024:
            assert part <= n * K * 4 * -(-nx // 64)
        assert part <= max(BOUND, 32 * ncb * nseg)
        assert (rounds == 1) == (n * K * ncb * nseg <= BOUND)
