"""The work split of the visibility sums (rt_visibility.hip, built for the host): it
depends on the image alone, so a point's sum is the same bits however many other
points a call asks for."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_05635_amd", "csrc")
SIZES = [(1, 1), (16, 16), (17, 300), (64, 255), (64, 256), (64, 257), (65, 1000), (128, 1024), (301, 187), (333, 777),
         (512, 512), (1024, 1024), (4096, 4096), (24, 8192), (8192, 24), (1 << 20, 3), (3, 1 << 20)]
POINTS = [1, 31, 32, 33, 64, 1024, 2000, 2048, 4097, 60000, 1 << 22]


@pytest.fixture(scope="module")
def layout(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("visibility") / "layout_driver")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=on",
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "visibility", "layout_driver.hip"),
                    os.path.join(CSRC, "rt_visibility.hip"), "-o", exe], check=True, capture_output=True)
    rows = np.array([(nx, ny, K) for nx, ny in SIZES for K in POINTS], dtype=np.int32)
    out = subprocess.run([exe], input=rows.tobytes(), capture_output=True, check=True).stdout
    return rows, np.frombuffer(out, dtype=np.int64).reshape(len(rows), -1)


def test_split_of_an_image(layout):
    _, out = layout
    per = out[:, :2].reshape(len(SIZES), len(POINTS), 2)
    assert (per == per[:, :1]).all()
