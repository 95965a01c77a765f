"""The function policies of rt_functions.h, built for the host: the pinned
coefficients give the direct functions' right-hand side bit for bit (the
kernels that pin them trace the rays the others trace)."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_05635_amd", "csrc")
SRC = os.path.join(HERE, "functions", "functions_driver.hip")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("functions") / "functions_driver")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=on",
                    "-I", CSRC, "-I", os.path.join(os.path.dirname(HERE), "include"), SRC, "-o", exe],
                   check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("metric", [0, 1, 2, 3])
def test_pinned_equals_direct(driver, metric):
    rng = np.random.default_rng(metric)
    n = 4000
    lam, lc, eta = rng.uniform(0.05, 0.3, n), rng.uniform(0.5, 30.0, n), rng.uniform(0.0, 0.34, n)
    m = (1.0 / lam, 0 * lam, 0 * lam) if metric == 1 else (lc, 1.0 / lc, eta * lc)
    R = np.concatenate([np.exp(rng.uniform(np.log(0.3), np.log(3000.0), n - 5)), [-2.0, 0.0, np.inf, np.nan, 1e-300]])
    th = np.concatenate([rng.uniform(-7.0, 7.0, n - 3), [0.0, np.pi / 2, np.nan]])
    rows = np.stack([np.full(n, float(metric)), rng.uniform(-1.0, 1.0, n), *m, rng.uniform(0.9, 1.1, n),
                     rng.uniform(-7.0, 7.0, n), R, th, rng.uniform(-2.0, 2.0, n), rng.uniform(-7.0, 7.0, n)], axis=1)
    out = subprocess.run([driver], input=rows.tobytes(), capture_output=True, check=True).stdout
    d = np.frombuffer(out).reshape(n, 2, 6)
    assert np.isfinite(d[:, 0]).all(axis=1).sum() > 0.98 * n
    same = d[:, 0].view(np.uint64) == d[:, 1].view(np.uint64)
    assert (same | (np.isnan(d[:, 0]) & np.isnan(d[:, 1]))).all()
