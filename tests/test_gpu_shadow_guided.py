"""Guided passes of the shadow boundary: their brackets are the bits that uniform
multisection (the search that counts attempts) ends with, over samples per
direction, tolerances down to the grid's own resolution, a direction count that
leaves a partly filled wavefront, and transitions near either end of the bracket."""

import math

import numpy as np
import pytest

from paper_2605_05635_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    # metric, halo, spin, directions, (b_lo, b_hi), b_tol
    ("kerr", (0.0, 0.0), 0.9, 17, (2.0, 9.0), 1e-10),
    ("cnfw", (0.02, 10.0), -0.6, 5, (1.0, 30.0), 3e-11),
    ("einasto", (0.15, 0.0), 0.4, 9, (2.0, 9.0), 1e-12),   # below the finest cell
    ("kerr", (0.0, 0.0), 0.0, 3, (5.1, 9.0), 1e-9),        # next to b_lo (27^.5 = 5.196)
    ("kerr", (0.0, 0.0), 0.0, 3, (2.0, 5.25), 1e-9),       # next to b_hi
    ("kerr", (0.0, 0.0), 0.0, 2, (2.0, 5.0), 1e-9),        # not in the bracket
    ("cnfw", (0.02, 10.0), 0.94, 4, (2.0, 9.0), 0.5),      # one pass
]


@pytest.mark.parametrize("samples", [16, 32, 64])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[4]}-{c[5]:g}")
def test_guided_brackets_are_multisections(case, samples):
    import torch

    from paper_2605_05635_amd import rt
    metric, halo, spin, n, (lo, hi), tol = case
    img = W.image(metric=metric, halo=halo, spin=spin, incl=math.radians(70.0))
    psi = np.arange(n) * 2.0 * np.pi / n + 0.3
    d = torch.tensor(np.stack([np.cos(psi), np.sin(psi)], 1), device="cuda")
    out, st = rt.shadow_boundary(img, d, lo, hi, tol, samples=samples)
    ref, ref_st = torch.empty_like(out), torch.empty_like(st)
    attempts = torch.zeros(n, dtype=torch.int64, device="cuda")
    print(f"[shadow] {case} samples {samples}", flush=True)
    rt.rt_shadow_boundary(rt.params_from(img), d, lo, hi, tol, ref, ref_st, attempts,
                          samples=samples)
    torch.cuda.synchronize()
    assert torch.equal(st, ref_st)
    assert torch.equal(out, ref)
    assert int(attempts.min()) > 0


@pytest.mark.parametrize("metric,halo,spin,incl,samples,max_attempts", [
    ("cnfw", (0.026591071355334964, 8.124849903947785), 0.3562084272295464, 0.4731523157197913, 32, 649),
    ("kerr", (0.0, 0.0), 0.13626928861037746, 2.903320946624731, 64, 416),
    ("cnfw", (0.16527745632976956, 10.842416819431184), -0.6794538286157996, 2.9009015502112625, 64, 492),
    ("einasto", (0.15, 0.0), 0.4, 1.2, 16, 250),
])
def test_rays_out_of_attempts(metric, halo, spin, incl, samples, max_attempts):
    """Rays that end by the attempt limit count as inside wherever they are, so which
    edges are sampled could decide; such directions go by uniform passes."""
    import torch

    from paper_2605_05635_amd import rt
    n = 200
    img = W.image(metric=metric, halo=halo, spin=spin, incl=incl, max_attempts=max_attempts)
    psi = (np.arange(n) + 0.3) * 2 * np.pi / n
    d = torch.tensor(np.stack([np.cos(psi), np.sin(psi)], 1), device="cuda")
    print(f"[shadow] {metric} samples {samples} max_attempts {max_attempts}", flush=True)
    out, st = rt.shadow_boundary(img, d, 2.0, 9.0, 1e-10, samples=samples)
    ref, ref_st = torch.empty_like(out), torch.empty_like(st)
    attempts = torch.zeros(n, dtype=torch.int64, device="cuda")
    rt.rt_shadow_boundary(rt.params_from(img), d, 2.0, 9.0, 1e-10, ref, ref_st, attempts, samples=samples)
    torch.cuda.synchronize()
    assert torch.equal(st, ref_st)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("tol,b_tol", [(1e-2, 1e-8), (1e-4, 1e-10), (2e-6, 1e-9), (1e-6, 1e-10), (1e-7, 1e-10)])
def test_loose_integrations(tol, b_tol):
    """Fates are out of order within the integration's error of the transition: loose
    ones are searched by uniform passes, and from 1e-7 down guided passes agree."""
    import torch

    from paper_2605_05635_amd import rt
    n = 300
    img = W.image(metric="cnfw", halo=(0.05, 8.0), spin=0.7, incl=1.1, rtol=tol, atol=tol)
    psi = (np.arange(n) + 0.3) * 2 * np.pi / n
    d = torch.tensor(np.stack([np.cos(psi), np.sin(psi)], 1), device="cuda")
    print(f"[shadow] tolerance {tol}", flush=True)
    out, st = rt.shadow_boundary(img, d, 2.0, 9.0, b_tol, samples=16)
    ref, ref_st = torch.empty_like(out), torch.empty_like(st)
    attempts = torch.zeros(n, dtype=torch.int64, device="cuda")
    rt.rt_shadow_boundary(rt.params_from(img), d, 2.0, 9.0, b_tol, ref, ref_st, attempts, samples=16)
    torch.cuda.synchronize()
    assert torch.equal(st, ref_st)
    assert torch.equal(out, ref)


@pytest.mark.parametrize("length", [2.0 ** -7, 1.0, 2.0 ** 10])
def test_direction_lengths(length):
    """b is in units of the direction's length; guided passes go by the impact parameter."""
    import torch

    from paper_2605_05635_amd import rt
    n = 100
    img = W.image(metric="cnfw", halo=(0.02, 10.0), spin=0.94, incl=1.2)
    psi = (np.arange(n) + 0.3) * 2 * np.pi / n
    d = torch.tensor(np.stack([np.cos(psi), np.sin(psi)], 1), device="cuda")
    print(f"[shadow] directions of length {length}", flush=True)
    ref, ref_st = torch.empty(n, 2, dtype=torch.float64, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    attempts = torch.zeros(n, dtype=torch.int64, device="cuda")
    rt.rt_shadow_boundary(rt.params_from(img), d, 2.0, 9.0, 1e-10, ref, ref_st, attempts, samples=16)
    out, st = rt.shadow_boundary(img, d * length, 2.0 / length, 9.0 / length, 1e-10 / length, samples=16)
    torch.cuda.synchronize()
    assert torch.equal(st, ref_st)
    assert torch.equal(out * length, ref)
