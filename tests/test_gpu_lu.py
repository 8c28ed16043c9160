"""The factorisation with the matrix in registers at the edges of its tiles and forms (64, 128, 192 and 256 rows,
the blocked form above): the form for up to 64 rows and the one for up to 128 do the same operations in the
same order, so a layer has the same bits by either; beyond 128 rows the per-order responses of a strongly
coupled layer are within 1e-9 of the layer's largest (the gate of the general solver)."""

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


def layer(N):
    return hg_like_coefficients(np.random.default_rng(700 + N), 40)[0], 1.7, 0.96


@pytest.mark.parametrize("N", [3, 4, 5, 8, 9, 12, 13, 15, 16])
def test_same_bits_beside_a_larger_layer(N):
    c, tau, om = layer(N)
    c2, tau2, om2 = layer(17)
    alone = BRDFSolver([N], [40], [4], [6])([tau], [om], [c])[0]
    beside = BRDFSolver([N, 17], [40, 40], [4, 2], [6, 6])([tau, tau2], [om, om2], [c, c2])[0]
    assert torch.equal(alone, beside)


@pytest.mark.parametrize("N", [17, 31, 32, 33, 36, 37, 47, 48, 49, 51, 63, 64, 65])
def test_sizes_against_oracle(N):
    c, tau, om = layer(N)
    s = BRDFSolver([N], [40], [2], [3])
    s([tau], [om], [c])
    _, Ro = dom.brdf(c, tau, om, N, 2, 3, return_orders=True)
    top = max(np.abs(R).max() for R in Ro)
    for m in range(2):
        assert np.abs(s.plan.inspect(0, m)[0] - Ro[m]).max() < 1e-9 * top, m
