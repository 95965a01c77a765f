"""The visibility summaries of Sec. 6.4 on the GPU (rt_visibility_dft, its
batched form, rt_visibility_rings) and the relative deviations of Sec. 6.2
(rt_relative_deviation), against the oracle's direct sums and closed forms.

Tolerance.  Both sides sum the same terms; the GPU takes its phases from a
recurrence re-seeded every 64 columns (relative error ~1e-14) and sums in a
different order, so V agrees with the direct sum to ~1e-14 of the flux: the
bar is 1e-11 of |V(0,0)| (amplitudes: 1e-11 absolute).  A batched call equals
the single-image calls bit for bit (the same work items per image).
"""
import math
import sys

import numpy as np
import pytest

from paper_2605_05635_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-11


@pytest.fixture(scope="module")
def rt():
    import torch
    assert torch.cuda.is_available(), "GPU test run without a GPU"
    from paper_2605_05635_amd import rt as mod
    return mod


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def ring_image(img, seed):
    rng = np.random.default_rng(seed)
    X = img["x_min"] + (np.arange(img["nx"]) + 0.5) * (img["x_max"] - img["x_min"]) / img["nx"]
    Y = img["y_min"] + (np.arange(img["ny"]) + 0.5) * (img["y_max"] - img["y_min"]) / img["ny"]
    rho = np.hypot(X[None, :] - 0.5, Y[:, None] + 0.3)
    I = np.exp(-0.5 * ((rho - 4.5) / 0.7) ** 2) * (1.0 + 0.4 * np.sin(1.3 * X[None, :]))
    return I + 0.05 * rng.random(I.shape)


SCREENS = [
    W.image(nx=97, ny=61, x_min=-10, x_max=10, y_min=-9, y_max=9),
    W.image(nx=1, ny=33, x_min=-1, x_max=1, y_min=-8, y_max=8),
    W.image(nx=40, ny=1, x_min=-8, x_max=8, y_min=-1, y_max=1),
    W.image(nx=128, ny=128),
    W.image(nx=200, ny=17, x_min=-12, x_max=13, y_min=-3, y_max=2),
]
KS = [2000, 1, 65, 300, 64]


def test_batch_equals_single_and_oracle(rt, orc):
    import torch
    say("[vis] 5 ragged screens: batch vs single vs oracle")
    imgs, Is, uvs = [], [], []
    for j, (img, K) in enumerate(zip(SCREENS, KS)):
        imgs.append(img)
        Is.append(torch.tensor(ring_image(img, j), device="cuda"))
        uvs.append(torch.tensor(W.uv_points(70 + j, K), device="cuda"))
    amps_b = [torch.empty(u.shape[0], dtype=torch.float64, device="cuda") for u in uvs]
    vis_b = [torch.empty(u.shape[0], 2, dtype=torch.float64, device="cuda") for u in uvs]
    rt.rt_visibility_dft_batch([rt.vis_image_from(i, I, u, a, v)
                                for i, I, u, a, v in zip(imgs, Is, uvs, amps_b, vis_b)])
    for img, I, uv, ab, vb in zip(imgs, Is, uvs, amps_b, vis_b):
        a1 = torch.empty_like(ab)
        v1 = torch.empty_like(vb)
        rt.rt_visibility_dft(I, rt.params_from(img), uv, amp=a1, vis=v1)
        torch.cuda.synchronize()
        assert torch.equal(a1, ab) and torch.equal(v1, vb)
        In, uvn = I.cpu().numpy(), uv.cpu().numpy()
        V = orc.visibility(img, In, uvn)
        F = abs(orc.flux_centroid(img, In)[0])
        vg = vb.cpu().numpy()
        assert np.abs(vg[:, 0] - V.real).max() <= TOL * F
        assert np.abs(vg[:, 1] - V.imag).max() <= TOL * F
        assert np.abs(ab.cpu().numpy() - np.abs(V) / F).max() <= TOL


def test_rings_closed_form_and_oracle(rt, orc):
    """V(q) and V(|u|, 0) of an elliptical Gaussian against their closed forms
    (exp(-pi^2 q^2 (sx^2 + sy^2)) I_0(pi^2 q^2 (sx^2 - sy^2)), exp(-2 pi^2 sx^2 q^2)),
    and of a traced image against the oracle's."""
    import torch
    from scipy.special import i0
    say("[vis] rings: elliptical Gaussian and a traced image")
    img = W.image(nx=150, ny=140, x_min=-12, x_max=12, y_min=-11, y_max=11)
    X = img["x_min"] + (np.arange(150) + 0.5) * 24 / 150
    Y = img["y_min"] + (np.arange(140) + 0.5) * 22 / 140
    sx, sy = 1.1, 0.6
    I = np.exp(-(X[None, :] + 0.3) ** 2 / (2 * sx * sx) - (Y[:, None] - 0.2) ** 2 / (2 * sy * sy))
    q = np.linspace(0.0, 0.45, 37)
    avg, cut = rt.visibility_rings(img, torch.tensor(I, device="cuda"), q, 48)
    avg, cut = avg.cpu().numpy(), cut.cpu().numpy()
    a, b = math.pi ** 2 * q ** 2 * (sx * sx + sy * sy), math.pi ** 2 * q ** 2 * (sx * sx - sy * sy)
    assert np.abs(avg - np.exp(-a) * i0(b)).max() <= 1e-10
    assert np.abs(cut - np.exp(-2 * math.pi ** 2 * sx * sx * q ** 2)).max() <= 1e-10
    timg = W.image(metric="cnfw", spin=0.95, halo=(0.02, 10.0), incl=math.radians(70), nx=96,
                   ny=90, x_min=-12, x_max=12, y_min=-12, y_max=12)
    outs = rt.trace(timg)
    qs = np.linspace(0.0, 0.5, 11)
    avg, cut = rt.visibility_rings(timg, outs["intensity"], qs, 24)
    torch.cuda.synchronize()
    oa, oc = orc.visibility_rings(timg, outs["intensity"].cpu().numpy(), qs, 24)
    assert np.abs(avg.cpu().numpy() - oa).max() <= TOL
    assert np.abs(cut.cpu().numpy() - oc).max() <= TOL


def test_batch_64_workload_sampled(rt, orc, batch64):
    """The benchmark's 64-image batch, traced as one launch, then its 2000
    visibilities per image in one batched call; 12 points of every image
    against the oracle's direct sum over the same image."""
    import torch
    imgs = batch64
    say("[vis] batch_64: trace + batched visibilities, 12 sampled points per image")
    many = rt.trace_many(imgs)
    uvs = [W.uv_points(1000 + j, 2000) for j in range(len(imgs))]
    amps = rt.visibility_many(imgs, [o["intensity"] for o in many], uvs)
    torch.cuda.synchronize()
    pick = np.arange(0, 2000, 167)
    for img, o, uv, amp in zip(imgs, many, uvs, amps):
        want = orc.visibility_amplitude(img, o["intensity"].cpu().numpy(), uv[pick])
        assert np.abs(amp.cpu().numpy()[pick] - want).max() <= TOL


def test_relative_deviation(rt, orc):
    import torch
    q = torch.tensor([1.0, 2.5, -3.0, 0.0, 7.0, 1e-300], dtype=torch.float64, device="cuda")
    r = torch.tensor([2.0, 2.5, 1.5, 4.0, 0.0, 3.0], dtype=torch.float64, device="cuda")
    d = rt.relative_to_reference(q, r).cpu().numpy()
    want = orc.relative_to_reference(q.cpu().numpy(), r.cpu().numpy())
    assert np.array_equal(d, want)
    # the diagnostics of two traced images, as the paper's table compares them
    base = dict(spin=0.95, incl=math.radians(70), nx=80, ny=80, x_min=-12, x_max=12, y_min=-12,
                y_max=12)
    kerr = W.image(metric="kerr", **base)
    cn = W.image(metric="cnfw", halo=(0.02, 10.0), **base)
    dk = rt.image_diagnostics(kerr, rt.trace(kerr)["intensity"], 0.1, 120)
    dc = rt.image_diagnostics(cn, rt.trace(cn)["intensity"], 0.1, 120)
    qk = torch.stack([dk[k] for k in rt.DIAG_KEYS])
    qc = torch.stack([dc[k] for k in rt.DIAG_KEYS])
    delta = rt.relative_to_reference(qc, qk).cpu().numpy()
    assert np.array_equal(delta, orc.relative_to_reference(qc.cpu().numpy(), qk.cpu().numpy()))


@pytest.mark.parametrize("nx,ny,K", [(1, 1, 1), (15, 8, 16), (16, 9, 17), (17, 7, 32), (63, 255, 33), (64, 256, 31),
                                     (65, 258, 2), (130, 519, 48), (8, 1031, 64)])
def test_tile_edges(rt, orc, nx, ny, K):
    """Screens and point counts around the edges of the kernel's tiles (16
    columns in blocks of 64, quads of folded rows in segments, 16 points in
    groups of 32), rings with an odd and an even number of angles."""
    import torch
    say(f"[vis] tile edges {nx} x {ny}, {K} points")
    img = W.image(nx=nx, ny=ny, x_min=-9, x_max=11, y_min=-8, y_max=7)
    I = torch.tensor(ring_image(img, nx + ny), device="cuda")
    uv = torch.tensor(W.uv_points(nx * ny, K), device="cuda")
    vis = torch.empty(K, 2, dtype=torch.float64, device="cuda")
    rt.rt_visibility_dft(I, rt.params_from(img), uv, vis=vis)
    In = I.cpu().numpy()
    V = orc.visibility(img, In, uv.cpu().numpy())
    flux = In.sum() * (20.0 / nx) * (15.0 / ny)
    got = vis.cpu().numpy()
    assert np.abs(got[:, 0] + 1j * got[:, 1] - V).max() <= TOL * flux
    q = np.linspace(0.0, 0.4, 3)
    for n_angles in (1, 2, 7, 12):
        avg, cut = rt.visibility_rings(img, I, q, n_angles)
        a, c = orc.visibility_rings(img, In, q, n_angles)
        assert np.abs(avg.cpu().numpy() - a).max() <= TOL
        assert np.abs(cut.cpu().numpy() - c).max() <= TOL


@pytest.mark.parametrize("nx,ny,many", [(64, 600, 140000), (130, 1030, 70000), (333, 260, 40000)])
def test_points_alone_and_among_many(rt, nx, ny, many):
    """A point's amplitude and visibility are the same bits however many others the call has."""
    import torch

    img = W.image(metric="kerr", nx=nx, ny=ny)
    I = torch.tensor(np.random.default_rng(nx).random((ny, nx)), device="cuda")
    uv = torch.tensor(np.random.default_rng(ny).uniform(-0.5, 0.5, (many, 2)), device="cuda")

    def run(points):
        amp = torch.empty(len(points), dtype=torch.float64, device="cuda")
        vis = torch.empty(len(points), 2, dtype=torch.float64, device="cuda")
        rt.rt_visibility_dft(I, rt.params_from(img), points, amp, vis)
        return amp, vis
    say(f"{nx}x{ny}, {many} points")
    amp, vis = run(uv)
    for k in (1, 33, 500):
        for first in (0, 5):
            a, v = run(uv[first:first + k].contiguous())
            assert torch.equal(a, amp[first:first + k]) and torch.equal(v, vis[first:first + k])


def test_rounds_of_many_points(rt):
    """More points than one round's scratch holds: the same bits as in calls of a few."""
    import torch

    img = W.image(metric="kerr", nx=70, ny=2100)
    I = torch.tensor(np.random.default_rng(7).random((2100, 70)), device="cuda")
    n = (1 << 24) // 18 + 100   # two column blocks, nine segments
    uv = torch.tensor(np.random.default_rng(8).uniform(-0.5, 0.5, (n, 2)), device="cuda")
    say(f"70x2100, {n} points")
    amp = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
    vis = torch.empty(n, 2, dtype=torch.float64, device="cuda")
    rt.rt_visibility_dft(I, rt.params_from(img), uv, amp, vis)
    assert float(amp.min()) >= 0.0
    for k in (0, n - 150, n // 2):
        a, v = torch.empty(150, dtype=torch.float64, device="cuda"), torch.empty(150, 2, dtype=torch.float64, device="cuda")
        rt.rt_visibility_dft(I, rt.params_from(img), uv[k:k + 150].contiguous(), a, v)
        assert torch.equal(a, amp[k:k + 150]) and torch.equal(v, vis[k:k + 150])
    # images that share a round with others, and one of a round of its own
    amps = rt.visibility_many([img, img, img], [I, I, I], [uv[:400000], uv, uv[5:900]])
    assert torch.equal(amps[0], amp[:400000]) and torch.equal(amps[1], amp) and torch.equal(amps[2], amp[5:900])
