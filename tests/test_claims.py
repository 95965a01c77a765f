"""The trace kernels' claims of tile parts (rt_ray.h, compiled for the host): every
pixel of a screen is handed out once, over tiles clipped at the edges, tiles of
one row and one column, claims that begin and end inside a tile, and any order in
which the wavefronts claim."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("claims") / "claim_driver")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "paper_2605_05635_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "tiles", "claim_driver.hip"), "-o", exe],
                   check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("nx,ny", [(1, 1), (8, 8), (9, 7), (64, 64), (301, 187), (37, 1), (1, 50)])
@pytest.mark.parametrize("tw,th", [(8, 8), (1, 1), (5, 3), (16, 6), (64, 2)])
def test_every_pixel_once(driver, nx, ny, tw, th):
    tw, th = min(tw, nx), min(th, ny)
    parts = 4 * (-(-nx // tw) * -(-ny // th))
    cases = [(nx, ny, tw, th, fine, waves, 7 * fine + waves)
             for fine in (0, 1, 4, parts // 3, parts, 1 << 40) for waves in (1, 3, 40)]
    out = subprocess.run([driver], input=np.array(cases, dtype=np.int64).tobytes(), capture_output=True,
                         check=True).stdout
    assert (np.frombuffer(out, dtype=np.int64).reshape(len(cases), nx * ny) == 1).all()
