"""Radial profile of the image diagnostics where a pixel centre lies on a bin's edge
or next to it, and at bin widths whose square leaves the normal range: each bin
holds the pixels with floor(sqrt(X^2 + Y^2) / bw) == k in IEEE arithmetic, one
rounding per operation (numpy's).  A bin's mean is then a sum of at most n
positive terms in another order, n 2^-53 relative."""

import numpy as np
import pytest

from paper_2605_05635_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,half,bw,bins", [
    (101, 101, 50.5, 1.0, 80),       # integer centres, integer edges (Pythagorean radii)
    (101, 101, 50.5, 0.2, 300),      # edges k * 0.2 that are not representable
    (1500, 40, 7.5, 0.01, 400),      # more columns than threads in a workgroup
    (30, 1500, 7.5, 1.0 / 3.0, 33),  # more rows
    (64, 64, 1.0, 1e-160, 3),        # (k bw)^2 underflows
    (64, 64, 1e150, 3e148, 40),      # and is near the top of the range
    (65, 65, 32.5, 1e200, 2),        # overflows; every pixel in bin 0
])
def test_bins_by_their_definition(nx, ny, half, bw, bins):
    import torch

    from paper_2605_05635_amd import rt
    hy = half * ny / nx
    img = W.image(nx=nx, ny=ny, x_min=-half, x_max=half, y_min=-hy, y_max=hy)
    I = np.random.default_rng(nx * ny).uniform(0.5, 1.5, (ny, nx))
    print(f"[diag] bins {nx}x{ny} bw {bw}", flush=True)
    got = rt.image_diagnostics(img, torch.tensor(I, device="cuda"), bw, bins)["profile"].cpu().numpy()
    dx, dy = (img["x_max"] - img["x_min"]) / nx, (img["y_max"] - img["y_min"]) / ny
    X = img["x_min"] + (np.arange(nx) + 0.5) * dx
    Y = img["y_min"] + (np.arange(ny) + 0.5) * dy
    with np.errstate(over="ignore"):
        k = np.floor(np.sqrt(X[None, :] * X[None, :] + Y[:, None] * Y[:, None]) / bw)
    n = np.array([(k == b).sum() for b in range(bins)])
    want = np.array([I[k == b].sum() / n[b] if n[b] else np.nan for b in range(bins)])
    assert np.array_equal(np.isnan(got), n == 0)
    ok = n > 0
    assert (np.abs(got[ok] / want[ok] - 1.0) <= (n[ok] + 2) * 2.0 ** -53 * 2).all()
