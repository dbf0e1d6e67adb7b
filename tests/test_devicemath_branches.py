"""The branches of the FP64 per-pair math that only the device build has (reciprocal
square root and Jacobi rotation from hardware estimates and Newton steps, with
range guards), compiled for the host with estimates of the accuracy that the
instructions state (2^29 units in the last place), at the guards and across
the range of doubles."""

import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_02080_amd", "csrc")

SOURCE = r"""
#include <math.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
static double err = 0.0;  // the estimates' relative error
static double est_rsq(double d) { return 1.0 / sqrt(d) * (1.0 + err); }
static double est_rcp(double d) { return 1.0 / d * (1.0 + err); }
#define __HIP_DEVICE_COMPILE__ 1
#define __builtin_amdgcn_rsq est_rsq
#define __builtin_amdgcn_rcp est_rcp
#include "dmath.h"
using namespace s3a;
extern "C" {
void set_err(double e) { err = e; }
double rsq(double d) { return rsqrt_pos(d); }
void rot(double app, double aqq, double apq, double* o) { jacobi_rotation(app, aqq, apq, o[0], o[1], o[2]); }
void sv3(const double* M, double* sv) { singular_values3(M, sv); }
void cross(const double* M, double* R) { rotation_from_cross_cov(M, R); }
int chol7(double* L, const double* b, double* x) { return cholesky_solve_packed<7>(L, b, x) ? 0 : 1; }
}
"""

ERR = 2.0 ** -23
EPS = 2.0 ** -53


@pytest.fixture(scope="module", params=[ERR, -ERR, 0.0])
def lib(request, tmp_path_factory):
    d = tmp_path_factory.mktemp("dmath")
    src, out = d / "t.cpp", d / "t.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + CSRC, "-o", str(out), str(src)], check=True)
    L = ctypes.CDLL(str(out))
    L.rsq.restype = ctypes.c_double
    L.rsq.argtypes = [ctypes.c_double]
    L.rot.argtypes = [ctypes.c_double] * 3 + [ctypes.c_void_p]
    L.set_err.argtypes = [ctypes.c_double]
    L.set_err(request.param)
    return L


def ptr(a):
    return ctypes.c_void_p(a.ctypes.data)


def test_reciprocal_square_root(lib):
    """Two Newton steps square the estimate's error twice (1.5 e^2, far below a
    rounding); what is left is the last step's few roundings."""
    rng = np.random.default_rng(1)
    edges = [1e-290, np.nextafter(1e-290, 1), np.nextafter(1e-290, 0), 1e290, np.nextafter(1e290, 0),
             np.nextafter(1e290, np.inf), 5e-324, 2.3e-308, 1.7e308, 1.0, 2.0, 4.0]
    for d in np.r_[edges, 10.0 ** rng.uniform(-307, 308, 2000)]:
        want = 1 / np.sqrt(np.longdouble(d))
        assert abs(np.longdouble(lib.rsq(d)) - want) <= 4 * EPS * want, d
    assert np.isinf(lib.rsq(0.0)) and lib.rsq(np.inf) == 0.0 and np.isnan(lib.rsq(np.nan)) and np.isnan(lib.rsq(-1.0))


def test_jacobi_rotation(lib):
    """The rotation diagonalises: c^2 + s^2 = 1, and the off-diagonal element that is left
    is a few roundings of the matrix, at scales on both sides of the guards."""
    rng = np.random.default_rng(2)
    for scale in [1e-160, 1e-141, 0.999e-140, 1.001e-140, 1e-100, 1.0, 1e100, 0.999e140, 1.001e140, 1e150]:
        for ratio in [0.0, 1e-16, 1e-8, 1e-3, 1.0, 1e3, 1e8, 1e16]:
            for sign in (1, -1):
                app, apq = scale * rng.uniform(0.5, 1), sign * scale * rng.uniform(0.5, 1)
                aqq = app + (1 if rng.random() < 0.5 else -1) * ratio * scale
                o = np.zeros(3)
                lib.rot(app, aqq, apq, ptr(o))
                t, c, s = o.astype(np.longdouble)
                assert abs(c * c + s * s - 1) <= 8 * EPS and abs(t) <= 1 + 8 * EPS
                left = (c * c - s * s) * np.longdouble(apq) + c * s * (np.longdouble(app) - np.longdouble(aqq))
                assert abs(left) <= 16 * EPS * max(abs(app), abs(aqq), abs(apq)), (scale, ratio, sign)


@pytest.mark.parametrize("scale", [1e-75, 1e-70, 1e-35, 1.0, 1e35, 1e70])
def test_decompositions(lib, scale):
    """Singular values and the rotation of 3 x 3 matrices whose Jacobi steps fall on either side
    of the guards."""
    rng = np.random.default_rng(3)
    for _ in range(50):
        U, V = (np.linalg.qr(rng.normal(size=(3, 3)))[0] for _ in range(2))
        if np.linalg.det(U) * np.linalg.det(V) < 0:
            U[:, 2] *= -1
        M = np.ascontiguousarray(scale * U @ np.diag([3.0, 2.0, 1.0]) @ V.T)
        sv, R = np.zeros(3), np.zeros(9)
        lib.sv3(ptr(M), ptr(sv))
        lib.cross(ptr(M), ptr(R))
        # eigenvalues of M^T M to a few roundings of the largest: sv 1 of 3 keeps 9 x that
        assert np.abs(np.sort(sv)[::-1] / scale - [3, 2, 1]).max() <= 200 * EPS
        assert np.abs(R.reshape(3, 3) - U @ V.T).max() <= 1e-13


@pytest.mark.parametrize("scale", [1e-295, 1e-290, 1e-150, 1.0, 1e150, 1e290, 1e295])
def test_packed_cholesky(lib, scale):
    """Pivots on both sides of the guards; and a matrix that is not positive definite."""
    rng = np.random.default_rng(4)
    A = rng.normal(size=(9, 7))
    H = A.T @ A + np.eye(7)
    b = rng.normal(size=7)
    x = np.zeros(7)
    L = np.ascontiguousarray((H * scale)[np.tril_indices(7)])
    assert lib.chol7(ptr(L), ptr(b), ptr(x)) == 0
    assert np.abs(x * scale - np.linalg.solve(H, b)).max() <= 1e-13 * np.linalg.cond(H)
    H[3, 3] = -1.0
    L = np.ascontiguousarray((H * scale)[np.tril_indices(7)])
    assert lib.chol7(ptr(L), ptr(b), ptr(x)) == 1
