"""The shadow boundary against multisection written out over traced screen points:
the first escaping edge of each level decides, in whatever order the fates beyond it
are.  Next to the polar axis the integration's error puts them out of order within
1e-5 M of the transition; at loose tolerances everywhere."""

import math

import numpy as np
import pytest

from paper_2605_05635_amd import workloads as W

pytestmark = pytest.mark.gpu

ESCAPED = 2
CASES = [
    # image, samples, tolerance, largest angle from the axis
    (dict(metric="cnfw", halo=(0.1522869694198339, 13.62397372197372), spin=-0.8954908840933054, incl=0.5289856452746222), 16, 1e-8, 1e-4),
    (dict(metric="kerr", halo=(0.0, 0.0), spin=-0.6864855241005801, incl=0.6271108759152196), 16, 1e-8, 1e-4),
    (dict(metric="einasto", halo=(0.10949624784737813, 0.0), spin=0.3820919864036876, incl=2.9255385797365987), 16, 1e-9, 1e-4),
    (dict(metric="kerr", halo=(0.0, 0.0), spin=-0.18933782942015054, incl=1.4925089468806474), 32, 1e-7, 1e-3),
    (dict(metric="einasto", halo=(0.16493212093304294, 0.0), spin=0.07208712435648601, incl=0.9383419185779497), 64, 1e-7, 1e-3),
    (dict(metric="cnfw", halo=(0.6, 8.0), spin=0.7, incl=1.1), 16, 1e-8, math.pi),
    (dict(metric="cnfw", halo=(0.05, 8.0), spin=0.7, incl=1.1), 32, 1e-5, math.pi),
    (dict(metric="kerr", halo=(0.0, 0.0), spin=0.9, incl=1.3), 16, 1e-4, math.pi),
]


def multisection(rt, img, d, lo, hi, tol, S):
    import torch
    lo = torch.full((len(d),), lo, dtype=torch.float64, device="cuda")
    hi = torch.full_like(lo, hi)
    j = torch.arange(1, S + 1, dtype=torch.float64, device="cuda")
    cells = torch.full_like(lo, S + 1.0)   # (a division by a number goes through its reciprocal)
    for _ in range(64):
        open_ = hi - lo > tol
        if not bool(open_.any()):
            break
        steps = j[None, :] * ((hi - lo) / cells)[:, None]
        edges = torch.cat([lo[:, None], lo[:, None] + steps, hi[:, None]], dim=1)
        xy = (edges[:, 1:-1, None] * d[:, None, :]).reshape(-1, 2).contiguous()
        out = rt.trace_points(img, xy, emission=False)["status"].reshape(len(d), S) == ESCAPED
        first = torch.where(out.any(1), out.int().argmax(1), torch.full_like(lo, S, dtype=torch.int64))
        nlo, nhi = edges.gather(1, first[:, None])[:, 0], edges.gather(1, first[:, None] + 1)[:, 0]
        lo, hi = torch.where(open_, nlo, lo), torch.where(open_, nhi, hi)
    return torch.stack([lo, hi], dim=1)


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]['metric']}-{c[1]}-{c[2]:g}-{c[3]:.0e}")
@pytest.mark.parametrize("count", [False, True])
def test_first_escaping_edge_decides(case, count):
    import torch

    from paper_2605_05635_amd import rt
    kw, samples, tol, angle = case
    n, b_hi = 600, 20.0 if kw["halo"][0] > 0.5 else 9.0
    r = np.random.default_rng(samples)
    off = 10.0 ** r.uniform(-9.0, math.log10(angle), n)
    psi = r.choice([-0.5, 0.5], n) * math.pi + r.choice([-1.0, 1.0], n) * off
    img = W.image(**kw, nx=16, ny=16, rtol=tol, atol=tol)
    d = torch.tensor(np.stack([np.cos(psi), np.sin(psi)], 1), device="cuda")
    out, st = torch.empty(n, 2, dtype=torch.float64, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    attempts = torch.zeros(n, dtype=torch.int64, device="cuda") if count else None
    print(f"[shadow] {kw['metric']} samples {samples} tolerance {tol:g}", flush=True)
    rt.rt_shadow_boundary(rt.params_from(img), d, 2.0, b_hi, 1e-10, out, st, attempts, samples=samples)
    assert int(st.max()) == 0
    assert torch.equal(out, multisection(rt, img, d, 2.0, b_hi, 1e-10, samples))
