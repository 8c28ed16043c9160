"""The eigensolver of systems held in LDS at the edges of its forms: blocks below the smallest multi-bulge
pass, 32 and 48 rows (4, 6 or 8 bulges), 64 rows (matrix in 8 or 32 registers, eigenvectors with T in LDS or
not, one or two lines per lane), ragged sizes and the largest. Strongly coupled orders of one layer against
the oracle: per-order responses within 1e-9 of the layer's largest, F_r within 1e-10 of its largest (I, I)
entry (the gates of the general solver); the schedules give the same bits."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dom
from paper_1707_05882_amd import binding
from paper_1707_05882_amd.api import BRDFSolver
from workloads.layers import hg_like_coefficients

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        raise RuntimeError("GPU tests need a ROCm device")
    binding.load()


@pytest.mark.parametrize("N", [3, 4, 5, 7, 8, 9, 12, 13, 16, 17, 18, 23, 31, 32])
def test_strong_orders_against_oracle(N):
    L, M = 40, 6
    coef = hg_like_coefficients(np.random.default_rng(500 + N), L)[0]
    tau, om = 2.5, 0.97
    s = BRDFSolver([N], [L], [M], [5])
    F = s([tau], [om], [coef])[0].clone()
    Fo, Ro = dom.brdf(coef, tau, om, N, M, 5, return_orders=True)
    assert np.abs(F.cpu().numpy() - Fo).max() < 1e-10 * np.abs(Fo[..., 0, 0]).max()
    top = max(np.abs(R).max() for R in Ro)
    for m in range(M):
        R, lam = s.plan.inspect(0, m)
        assert np.abs(R - Ro[m]).max() < 1e-9 * top, m
        im = lam.imag[lam.imag != 0.0]
        assert np.array_equal(im[::2], -im[1::2])
    for sched in (binding.EIGEN_LONGEST_FIRST, binding.EIGEN_PERSISTENT):
        s.plan.set_tuning(sched, 16)
        assert torch.equal(s([tau], [om], [coef])[0], F)
