"""The shadow boundary's decisions (rt_search.h, compiled for the host) on scripted
rays, against multisection written out: the first escaping edge of each level."""
import os
import struct
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
M64 = (1 << 64) - 1


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("search") / "search_driver")
    subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=on",
                    "-I", os.path.join(ROOT, "paper_2605_05635_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "search", "search_driver.hip"), "-o", exe],
                   check=True, capture_output=True)

    def run(rows):
        rows = np.ascontiguousarray(rows, dtype=np.float64)
        out = subprocess.run([exe], input=rows.tobytes(), capture_output=True, check=True).stdout
        return np.frombuffer(out).reshape(len(rows), 7)
    return run


def hashed(x, seed):
    z = (struct.unpack("<Q", struct.pack("<d", x))[0] + seed * 0x9e3779b97f4a7c15) & M64
    z = ((z ^ (z >> 30)) * 0xbf58476d1ce4e5b9) & M64
    z = ((z ^ (z >> 27)) * 0x94d049bb133111eb) & M64
    return ((z ^ (z >> 31)) >> 11) * 2.0 ** -53


def escapes(row, b):
    b_c, jump, period, lost, seed = row[4:9]
    d, seed = b - b_c, int(seed)
    out = d > jump * (2.0 * hashed(float(np.floor(d / period)), seed) - 1.0)
    return out and not (abs(d) < lost and hashed(b, seed + 1) < 0.25)


def multisection(row):
    S, lo, hi, tol = row[:4]
    S = int(S)
    for _ in range(64):
        w = (hi - lo) / (S + 1)
        edges = [lo] + [lo + j * w for j in range(1, S + 1)] + [hi]
        first = next((j for j in range(1, S + 1) if escapes(row, edges[j])), S + 1)
        if (edges[first - 1], edges[first]) == (lo, hi):
            break
        lo, hi = edges[first - 1], edges[first]
        if not hi - lo > tol:
            break
    return lo, hi


def rows(S, n, b_tol, jump=0.0, period=1.0, lost=0.0):
    r = np.random.default_rng(S)
    return np.stack([np.full(n, float(S)), np.full(n, 2.0), np.full(n, 9.0), np.full(n, b_tol), r.uniform(2.5, 8.5, n),
                     np.full(n, jump), np.full(n, period), np.full(n, lost), np.arange(n) * 2.0, np.ones(n)], axis=1)


@pytest.mark.parametrize("S", [16, 32, 64])
@pytest.mark.parametrize("b_tol", [1e-4, 1e-10, 2e-12])
def test_in_order(driver, S, b_tol):
    """Fates in order: multisection's brackets, in fewer passes than its levels."""
    a = rows(S, 300, b_tol)
    d = driver(a)
    assert [tuple(x) for x in d[:, :2]] == [multisection(x) for x in a]
    assert not d[:, 4].any()
    if b_tol == 1e-10:
        assert d[:, 2].max() < np.ceil(np.log(7.0 / b_tol) / np.log(S + 1.0))


@pytest.mark.parametrize("S", [16, 32, 64])
@pytest.mark.parametrize("jump,period,lost", [(1e-9, 1e-9, 0.0), (1e-8, 3e-9, 0.0), (1e-7, 1e-7, 0.0), (1e-6, 3e-7, 0.0),
                                              (1e-5, 1e-5, 0.0), (1e-4, 1e-4, 0.0), (1e-3, 1e-3, 0.0), (0.0, 1.0, 1e-6),
                                              (0.0, 1.0, 1e-3), (1e-8, 1e-8, 1e-2),
                                              (1e-6, 1e-9, 0.0), (1e-4, 1e-7, 0.0)])
def test_out_of_order(driver, S, jump, period, lost):
    """The ray at a bracket's lower end ends inside and the one at its upper end
    escapes; a direction seen to be out of order ends with multisection's bracket,
    whatever guided passes before had settled, or multisection's is decided by an edge
    beyond the range in which those that they left out were traced."""
    a = rows(S, 1500, 1e-10, jump, period, lost)
    d = driver(a)
    seen = d[:, 4] != 0
    assert seen.sum() > 20
    assert not any(escapes(x, y) for x, y in zip(a, d[:, 0])) and all(escapes(x, y) for x, y in zip(a, d[:, 1]))
    ref = np.array([multisection(x) for x in a[seen]])
    same = (d[seen, :2] == ref).all(axis=1)
    assert (same | (ref[:, 1] < d[seen, 5]) | (ref[:, 0] > d[seen, 6])).all()
    assert same.all() or jump > 100 * period   # (hundreds of shifts within their own size)


@pytest.mark.parametrize("S", [16, 64])
@pytest.mark.parametrize("length", [2.0 ** -7, 2.0 ** 10])
def test_direction_length(driver, S, length):
    """b is in units of the direction's length: the same rays in the same passes."""
    a = rows(S, 300, 1e-10)
    scaled = a.copy()
    scaled[:, 1:5] /= length
    scaled[:, 9] = length
    d, e = driver(a), driver(scaled)
    assert np.array_equal(d[:, :2], e[:, :2] * length)
    assert np.array_equal(d[:, 2:5], e[:, 2:5])
