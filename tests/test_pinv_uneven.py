"""The truncated pseudo-inverse solve of the input estimation on matrices whose
rows differ in size, as those of records of unequal amplitude and of late
shifts do: no further off than the general path (the eigen-decomposition by
Jacobi rotations) is."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2404_17754_amd", "csrc")
P = C.POINTER(C.c_double)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("pinv") / "libpinv_check.so"
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, os.path.join(HERE, "pinv_check.cpp"),
                    os.path.join(HERE, "linalg_check.cpp"), "-o", str(out)], check=True)
    return C.CDLL(str(out))


def _solve(entry, a, h, cut):
    t = np.full(len(h), np.nan)
    kept = entry(len(h), a.ctypes.data_as(P), h.ctypes.data_as(P), t.ctypes.data_as(P), C.c_double(cut))
    return kept, t


# binary powers for the rows' sizes, so that the scaled matrix is exact; the
# ratio of the diagonal is 4 ** bits; every eigenvalue lies above the cut
@pytest.mark.parametrize("n", [3, 6, 12, 45, 150])
@pytest.mark.parametrize("bits", [0, 1, 2, 4, 7, 10, 14])
@pytest.mark.parametrize("order", ["falling", "rising", "blocks", "mixed"])
def test_rows_of_unequal_size(lib, n, bits, order):
    rng = np.random.default_rng(n + bits)
    g = rng.standard_normal((n, 4 * n))
    b = g @ g.T / (4 * n)                       # condition about 9
    b = (b + b.T) / 2
    k = {"falling": np.arange(n), "rising": np.arange(n)[::-1], "blocks": np.arange(n) * 3 // n * (n // 2),
         "mixed": rng.permutation(n)}[order]
    d = 2.0 ** -np.round(bits * np.minimum(k / (n - 1), 1.0))
    a, h = np.ascontiguousarray(b * d[:, None] * d), rng.standard_normal(n)
    kept, t = _solve(lib.pinv, a, np.ascontiguousarray(h * d), 2e-12)
    general, tg = _solve(lib.tsolve, a, np.ascontiguousarray(h * d), 2e-12)
    assert kept == general
    if kept < n:
        assert np.array_equal(t, tg)            # past the rule: the general path itself
        return
    want = np.linalg.solve(b, h) / d
    # twice the general path's error, or the rounding of n unknowns on the
    # scaled matrix (the reference's own solve included)
    floor = 20 * n ** 0.5 * np.finfo(float).eps * np.linalg.cond(b) * np.linalg.norm(want)
    assert np.linalg.norm(t - want) <= max(2 * np.linalg.norm(tg - want), floor)


def test_rows_of_zeros(lib):
    """Shifts past the last arrival: rows of zeros, their unknowns zero."""
    rng = np.random.default_rng(0)
    g = rng.standard_normal((20, 80))
    a = np.zeros((30, 30))
    a[5:25, 5:25] = g @ g.T
    h = np.zeros(30)
    h[5:25] = rng.standard_normal(20)
    kept, t = _solve(lib.pinv, a, h, 1e-6)
    assert kept == 20 and not t[:5].any() and not t[25:].any()
    assert np.allclose(t[5:25], np.linalg.solve(g @ g.T, h[5:25]), rtol=1e-12, atol=0)


def _exact(b, d, h):
    """Solution of (d b d) x = d h in extended precision (Cholesky of b)."""
    n = len(h)
    l = np.zeros((n, n), np.longdouble)
    b = b.astype(np.longdouble)
    for j in range(n):
        l[j, j] = np.sqrt(b[j, j] - l[j, :j] @ l[j, :j])
        l[j + 1:, j] = (b[j + 1:, j] - l[j + 1:, :j] @ l[j, :j]) / l[j, j]
    y = h.astype(np.longdouble)
    for j in range(n):
        y[j] = (y[j] - l[j, :j] @ y[:j]) / l[j, j]
    for j in range(n - 1, -1, -1):
        y[j] = (y[j] - l[j + 1:, j] @ y[j + 1:]) / l[j, j]
    return y / d


@pytest.mark.parametrize("order", ["falling", "rising"])
def test_no_further_off_on_the_whole(lib, order):
    """Rows that fall or rise by up to the ratio that still takes the fast way:
    the geometric mean of the errors is no larger than the general path's."""
    ratio = []
    for n in (12, 20, 36, 64):
        bits = int(np.floor(np.log2(n / 2) / 2))   # largest power of 4 up to n / 2
        for seed in range(25):
            rng = np.random.default_rng(1000 * n + seed)
            g = rng.standard_normal((n, 4 * n))
            b = g @ g.T
            b = (b + b.T) / 2
            b /= np.sqrt(np.outer(np.diag(b), np.diag(b)))
            b = (b + b.T) / 2
            np.fill_diagonal(b, 1.0)
            k = np.arange(n) if order == "falling" else np.arange(n)[::-1]
            d = 2.0 ** -np.round(bits * k / (n - 1))
            h = rng.standard_normal(n)
            a, r = np.ascontiguousarray(b * d[:, None] * d), np.ascontiguousarray(h * d)
            want = _exact(b, d, h)
            err = [float(np.linalg.norm(_solve(f, a, r, 1e-6)[1] - want)) for f in (lib.pinv, lib.tsolve)]
            assert not np.array_equal(_solve(lib.pinv, a, r, 1e-6)[1], _solve(lib.tsolve, a, r, 1e-6)[1])
            ratio.append(err[0] / err[1])
    print(order, np.exp(np.mean(np.log(ratio))), max(ratio))
    assert np.exp(np.mean(np.log(ratio))) <= 1.0
