"""The 4 x 4 eigen-decomposition of a node's Stokes block (csrc/eig4.hpp), compiled for the host: A Q = Q
Lambda in the eigensolver's storage (a complex pair as real and imaginary part) to a residual of
1e-11 |A|, which leaves room for blocks whose eigenvectors are close to dependent (a backward error of a
few 1e-16 grows with their condition, at most 1e6 by the determinant test)."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_1707_05882_amd", "csrc")


@pytest.fixture(scope="module")
def eig4(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("eig4")
    src = d / "eig4.cpp"
    src.write_text('#include "eig4.hpp"\nextern "C" int run(double* H, double* Q, double* wr, double* wi, double noise)'
                   "{ double X[32]; return vbrdf::eig4(H, Q, X, wr, wi, noise); }\n")
    so = d / "eig4.so"
    subprocess.run([cxx, "-O2", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    f = ctypes.CDLL(str(so)).run
    f.argtypes = [ctypes.c_void_p] * 4 + [ctypes.c_double]

    def call(A, noise):
        H, Q, wr, wi = A.copy(), np.zeros((4, 4)), np.zeros(4), np.zeros(4)
        ok = f(H.ctypes.data, Q.ctypes.data, wr.ctypes.data, wi.ctypes.data, noise)
        return bool(ok), Q, wr, wi

    return call


def _draw(rng, kind):
    A = rng.standard_normal((4, 4))
    if kind == "symmetric":
        return A + A.T
    if kind == "scaled":
        return A * 10.0 ** rng.uniform(-200, 100)
    if kind == "sparse":
        A[rng.random((4, 4)) < 0.5] = 0.0
        return A
    if kind == "stokes":  # symmetric but for the antisymmetric U-V coupling, I-Q and U-V loosely coupled
        S = A + A.T
        S[2, 3] = -S[3, 2]
        S[:2, 2:] *= 1e-3
        S[2:, :2] *= 1e-3
        return S * 1e-9
    return A


@pytest.mark.parametrize("kind", ["general", "symmetric", "scaled", "sparse", "stokes"])
def test_residual(eig4, kind):
    rng = np.random.default_rng(17)
    refused = 0
    for _ in range(4000):
        A = _draw(rng, kind)
        scale = np.abs(A).max()
        ok, Q, wr, wi = eig4(A, 2e-15 * scale)
        if not ok:  # only where the eigenvectors are dependent
            refused += 1
            assert abs(np.linalg.det(np.linalg.eig(A)[1])) < 1e-5
            continue
        L = np.diag(wr)
        for j in range(4):
            if wi[j] > 0:
                assert wr[j + 1] == wr[j] and wi[j + 1] == -wi[j]
                L[j, j + 1], L[j + 1, j] = wi[j], -wi[j]
        assert np.abs(A @ Q - Q @ L).max() < 1e-11 * scale
    assert refused < (4000 if kind == "sparse" else 4)


def test_special_blocks(eig4):
    for A in (np.zeros((4, 4)), np.diag([1.0, 2.0, 3.0, 4.0]), 5.0 * np.eye(4)):
        ok, Q, wr, wi = eig4(A, 0.0)
        assert ok and np.array_equal(Q, np.eye(4)) and np.array_equal(wr, np.diag(A)) and not wi.any()
    J = np.diag([1.0, 1.0, 2.0, 3.0])
    J[0, 1] = 1.0
    assert not eig4(J, 1e-15)[0]  # defective
    assert not eig4(np.full((4, 4), np.nan), 0.0)[0]
