"""The truncated pseudo-inverse solve of the input estimation
(sym_pinv_solve, csrc/sw_linalg.h) on the CPU against known spectra: every
size at which its reductions start, truncated, repeated and zero eigenvalues,
matrices that are tridiagonal or split already, and values that are not
finite."""
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
def pinv(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = tmp_path_factory.mktemp("pinv") / "libpinv_check.so"
    subprocess.run([gxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, os.path.join(HERE, "pinv_check.cpp"),
                    "-o", str(out)], check=True)
    lib = C.CDLL(str(out))
    lib.pinv.restype = C.c_int

    def solve(a, h, cut):
        a, h = np.ascontiguousarray(a, float), np.ascontiguousarray(h, float)
        t = np.full(len(h), np.nan)
        kept = lib.pinv(len(h), a.ctypes.data_as(P), h.ctypes.data_as(P), t.ctypes.data_as(P), C.c_double(cut))
        return kept, t
    return solve


def _check(pinv, q, lam, cut, rng):
    h = rng.standard_normal(len(lam))
    kept, t = pinv((q * lam) @ q.T, h, cut)
    keep = lam > cut * lam.max()
    assert kept == keep.sum()
    want = (q[:, keep] / lam[keep]) @ (q[:, keep].T @ h)
    kappa = lam.max() / lam[keep].min()
    # backward error eps of the reduction, times its size, on an operator of
    # norm 1 / lam_min and condition kappa (the right-hand side's part outside
    # the kept directions comes in through their rotation)
    size = np.linalg.norm(h) / lam[keep].min()
    assert np.linalg.norm(t - want) <= 8 * len(lam) ** 0.5 * np.finfo(float).eps * kappa * size


# spreads that put no eigenvalue on a cut, where rounding decides
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 12, 45, 150, 384])
@pytest.mark.parametrize("spread,cut", [(2.03, 1e-6), (9.13, 1e-6), (9.13, 1e-3), (14.21, 1e-11), (6.07, 0.5)])
def test_spread_spectra(pinv, n, spread, cut):
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = 3.0 * 10.0 ** -(spread * (np.arange(n) + 0.37) / n)
    _check(pinv, q, lam, cut, rng)


def test_repeated_negative_and_zero_eigenvalues(pinv):
    rng = np.random.default_rng(1)
    q, _ = np.linalg.qr(rng.standard_normal((20, 20)))
    for lam in (np.ones(20), np.repeat([4.0, 1.0], 10), np.r_[np.ones(15), np.zeros(5)], np.r_[np.ones(15), -np.ones(5)]):
        _check(pinv, q, lam, 1e-6, rng)
    assert pinv(np.zeros((7, 7)), rng.standard_normal(7), 1e-6)[0] == 0
    kept, t = pinv(-np.eye(6), np.ones(6), 1e-6)
    assert kept == 0 and np.all(t == 0)


def test_structured_matrices(pinv):
    rng = np.random.default_rng(2)
    h = rng.standard_normal(9)
    d = np.diag(np.arange(1.0, 10.0))
    assert np.allclose(pinv(d, h, 1e-6)[1], h / np.arange(1.0, 10.0), rtol=1e-14)
    tri = 4 * np.eye(9) + np.diag(np.ones(8), 1) + np.diag(np.ones(8), -1)
    assert np.allclose(pinv(tri, h, 1e-6)[1], np.linalg.solve(tri, h), rtol=1e-13)
    blocks = tri.copy()
    blocks[4, 5] = blocks[5, 4] = 0
    assert np.allclose(pinv(blocks, h, 1e-6)[1], np.linalg.solve(blocks, h), rtol=1e-13)
    for scale in (1e-200, 1e150):
        assert np.allclose(pinv(tri * scale, h * scale, 1e-6)[1], np.linalg.solve(tri, h), rtol=1e-13)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_values_that_are_not_finite_end(pinv, bad):
    a = 4 * np.eye(6)
    a[2, 3] = a[3, 2] = bad
    pinv(a, np.ones(6), 1e-6)
    pinv(4 * np.eye(6), np.r_[np.ones(5), bad], 1e-6)
