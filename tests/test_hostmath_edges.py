"""The FP64 per-pair math at the edges of its branches (host build): Exp where
its series change, the closed form on both sides of its degeneracy test."""

import ctypes
import os

import numpy as np
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_02080_amd", "libs3a_hostmath.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2510_02080_amd import build
        build.build()
    return ctypes.CDLL(LIB)


def expm_long(G):
    """exp of a 4x4 matrix in extended precision (scipy's expm is good to 5e-13 only near sigma = 4)."""
    A = G.astype(np.longdouble) / np.longdouble(2**10)
    P = np.eye(4, dtype=np.longdouble)
    E = P.copy()
    for n in range(1, 30):
        P = P @ A / np.longdouble(n)
        E = E + P
    for _ in range(10):
        E = E @ E
    return E


def dp(a):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


@pytest.mark.parametrize("sigma", [0.0, 1e-9, 0.0624999, 0.0625001, -0.0624999, -0.0625001, 0.3, 3.999, 4.001])
@pytest.mark.parametrize("theta", [0.0, 1e-7, 0.0999999, 0.1000001, 1.5])
def test_exp_series_edges(lib, sigma, theta):
    """Against the 4x4 matrix exponential: a handful of roundings of values of size e^sigma."""
    w = theta * np.array([2.0, -1.0, 2.0]) / 3.0
    xi = np.concatenate([[0.7, -1.3, 0.4], w, [sigma]])
    T = np.zeros(13)
    lib.s3a_host_sim3_exp(dp(xi), dp(T))
    G = np.zeros((4, 4))
    G[:3, :3] = np.array([[sigma, -w[2], w[1]], [w[2], sigma, -w[0]], [-w[1], w[0], sigma]])
    G[:3, 3] = xi[:3]
    E = expm_long(G)
    scale = max(1.0, np.exp(sigma))
    assert np.abs(T[12] * T[:9].reshape(3, 3) - E[:3, :3]).max() <= 2e-14 * scale
    assert np.abs(T[9:12] - E[:3, 3]).max() <= 2e-14 * scale


@pytest.mark.parametrize("ratio,ok", [(1.0, True), (1e-2, True), (1.7e-3, True), (1e-4, True), (1.1e-5, True), (0.9e-5, False), (0.0, False)])
def test_umeyama_second_singular_value(lib, ratio, ok):
    """Cross-covariances whose second singular value is `ratio` of the first: the
    rotation is found exactly where the test passes, refused below 1e-5."""
    rng = np.random.default_rng(5)
    U, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    V, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    U, V = U * np.sign(np.linalg.det(U)), V * np.sign(np.linalg.det(V))
    M = U @ np.diag([1.0, ratio, 0.5 * ratio]) @ V.T
    m = np.concatenate([[1.0], np.zeros(6), [3.0], M.ravel()])
    T = np.zeros(13)
    status = lib.s3a_host_umeyama(dp(m), dp(T))
    assert status == (0 if ok else 2)
    if ok:
        # U V^T; the eigenvector's error is the rounding of M over the gap of its quaternion form
        assert np.abs(T[:9].reshape(3, 3) - U @ V.T).max() <= 1e-14 / ratio


@pytest.mark.parametrize("xi", [
    np.zeros(7), [0, 0, 0, 0, 0, 0, 0.5], [0.4, -2.0, 1.0, 0, 0, 0, 0], [0.3, 0.1, -0.2, 1e-9, 0, 0, 1e-9],
    [0.7, -1.3, 0.4, 0.2, -0.1, 0.3, 0.1], [5.0, 8.0, -3.0, 1.9, -1.7, 1.8, -2.0], [20.0, 0, 0, 0, 3.0, 0, 4.0]])
def test_left_jacobian_transposed_on_a_vector(lib, xi):
    """J_l(xi)^T g by the vector series against the series in extended precision:
    roundings of terms that add up to at most e^|ad| times |g|."""
    xi = np.asarray(xi, dtype=np.float64)
    hat = lambda v: np.array([[0, -v[2], v[1]], [v[2], 0, -v[0]], [-v[1], v[0], 0]])
    A = np.zeros((7, 7))
    A[:3, :3] = hat(xi[3:6]) + xi[6] * np.eye(3)
    A[:3, 3:6], A[3:6, 3:6], A[:3, 6] = hat(xi[:3]), hat(xi[3:6]), -xi[:3]
    A = A.T.astype(np.longdouble)
    for g in list(np.eye(7)) + [np.random.default_rng(3).normal(size=7)]:
        term, want, size = g.astype(np.longdouble), g.astype(np.longdouble), np.abs(g).astype(np.longdouble)
        mag = size.copy()
        for n in range(1, 150):
            term, size = A @ term / (n + 1), np.abs(A) @ size / (n + 1)
            want, mag = want + term, mag + size
        out = np.zeros(7)
        lib.s3a_host_sim3_jacobian_t_apply(dp(xi), dp(np.ascontiguousarray(g)), dp(out))
        # term n carries at most 8 roundings a step; the terms that count end by n = 60
        assert (np.abs(out - want) <= 60 * 8 * 2.0**-53 * mag + 1e-17).all(), (g, out, want)
