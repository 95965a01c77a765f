"""Functions of the headers on the device, bit for bit: the square root without
range scaling against the device's IEEE one, and the policies of rt_functions.h
(coefficients pinned in registers, or taken through scalar registers) against the
direct functions, where a host build takes other instructions."""
import ctypes as C
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def ptr(t):
    return C.c_void_p(t.data_ptr())


def same_bits(a, b):
    return (a.view(np.uint64) == b.view(np.uint64)) | (np.isnan(a) & np.isnan(b))


def test_square_root(device_checks):
    import torch
    r = np.random.default_rng(1)
    n = 400000
    x = np.ldexp(r.uniform(1.0, 2.0, n), r.integers(-767, 1024, n))
    # squares and what lies next to them, where the rounding is closest
    s = np.ldexp(r.uniform(1.0, 2.0, n), r.integers(-383, 511, n)) ** 2
    x = np.concatenate([x, s, np.nextafter(s, np.inf), np.nextafter(s, 0.0),
                        [0.0, -0.0, np.inf, np.nan, -1.0, -np.inf, 2.0 ** -767, np.finfo(np.float64).max, 1.0, 4.0]])
    d = torch.tensor(x, device="cuda")
    fast, ieee = torch.empty_like(d), torch.empty_like(d)
    print(f"[functions] {len(x)} square roots", flush=True)
    assert device_checks.check_sqrt(ptr(d), ptr(fast), ptr(ieee), len(x)) == 0
    torch.cuda.synchronize()
    fast, ieee = fast.cpu().numpy(), ieee.cpu().numpy()
    with np.errstate(invalid="ignore"):
        assert same_bits(ieee, np.sqrt(x)).all()
    assert same_bits(fast, ieee).all()


@pytest.mark.parametrize("metric,m", [(0, (0.0, 0.0, 0.0)), (1, (1.0 / 0.14, 0.0, 0.0)), (1, (1.0 / 3.0, 0.0, 0.0)),
                                      (2, (8.0, 1.0 / 8.0, 0.6 * 8.0)), (2, (0.3, 1.0 / 0.3, 2.0 * 0.3)),
                                      (3, (10.0, 0.1, 0.02 * 10.0)), (3, (4.0, 0.25, 0.3 * 4.0))])
def test_policies(device_checks, metric, m):
    import torch
    r = np.random.default_rng(metric)
    n = 100000
    R = np.exp(r.uniform(math.log(0.3), math.log(3000.0), n))
    th = r.uniform(-7.0, 7.0, n)
    x = np.where(r.random(n) < 0.5, r.uniform(-3.0, 3.0, n), r.uniform(-800.0, 800.0, n))
    u = np.where(r.random(n) < 0.5, r.uniform(-0.999, 3.0, n), r.normal(0.0, 1.0, n) * 10.0 ** r.uniform(-18.0, -1.0, n))
    u[::5] = 10.0 ** r.uniform(0.0, 6.0, len(u[::5]))
    rows = torch.tensor(np.stack([R, th, x, u], axis=1), device="cuda")
    out = torch.empty(n, 3, 10, dtype=torch.float64, device="cuda")
    print(f"[functions] metric {metric} {m}", flush=True)
    assert device_checks.check_policies(metric, C.c_double(0.7), (C.c_double * 3)(*m), ptr(rows), ptr(out), n) == 0
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.isfinite(out[:, 0, [0, 1, 2, 3, 5]]).all()
    for policy in (1, 2):
        assert same_bits(out[:, 0], out[:, policy]).all(), policy
