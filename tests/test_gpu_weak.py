"""The iteration for weakly coupled orders: plans with enough orders to run it, at the edges of its tiles
and panels, against the oracle (F_r within 1e-10 of its largest (I, I) entry, per-order responses within
1e-9 of the layer's largest, as for the general solver), and an order in which the general solver fails."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dom
from oracle.quadrature import double_gauss
from paper_1707_05882_amd import binding
from paper_1707_05882_amd.api import BRDFSolver
from workloads.layers import hg_like_coefficients

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        raise RuntimeError("GPU tests need a ROCm device")
    binding.load()


# fewer rows than a tile (one or two nodes do not resolve these phase functions); a whole tile; one node more; ragged; one panel and two; the largest
# size taken whole; the smallest and a ragged size of which the faint orders are taken
@pytest.mark.parametrize("N,L,M", [(3, 24, 20), (4, 24, 20), (5, 24, 20), (13, 26, 22), (16, 32, 24),
                                   (17, 32, 24), (31, 48, 30), (32, 64, 40), (33, 66, 60), (45, 90, 80)])
def test_many_orders_against_oracle(N, L, M):
    nl = 256 // M + 1  # more than 256 orders
    rng = np.random.default_rng(1000 + N)
    coefs = [hg_like_coefficients(rng, L)[0] for _ in range(nl)]
    tau = 10.0 ** rng.uniform(-0.5, 1.5, nl)
    om = rng.uniform(0.6, 0.999, nl)
    s = BRDFSolver([N] * nl, [L] * nl, [M] * nl, [5] * nl)
    F = s(tau, om, coefs)
    for l in {0, nl - 1}:
        Fo, Ro = dom.brdf(coefs[l], tau[l], om[l], N, M, 5, return_orders=True)
        assert np.abs(F[l].cpu().numpy() - Fo).max() < 1e-10 * np.abs(Fo[..., 0, 0]).max()
        top = max(np.abs(R).max() for R in Ro)
        for m in range(0, M, 3):
            if 4 * N > 128 and np.abs(Ro[m]).max() > 1e-7 * top:
                continue  # above n = 128 the general solver's order, not the iteration's
            R, _ = s.plan.inspect(l, m)
            assert np.abs(R - Ro[m]).max() < 1e-9 * top, m


def test_order_in_which_the_general_solver_fails():
    """N = 48, order 87: the scattering is down to 1e-20 there, R^m is rounding noise, and the general
    solver's eigenvectors of the nearly fourfold eigenvalues came out dependent (R^m up to 7e10)."""
    N, L, M = 48, 96, 96
    l = np.arange(L)
    base = (2 * l + 1) * 0.5794274783833541 ** l
    hi = base * (l >= 2)
    rho, rho4, eta, zeta = 0.6369825046711112, 0.5558410980633085, 0.21777389720087598, 0.012480376474742228
    coef = np.stack([base, rho * hi, rho * hi, rho4 * base, -eta * hi, zeta * hi])
    tau, om = 2.9871358703417976, 0.5160563562786256
    s = BRDFSolver([N] * 3, [L] * 3, [M] * 3, [5] * 3)
    s([tau] * 3, [om] * 3, [coef] * 3)
    mu, alpha = double_gauss(N)
    top = np.abs(s.plan.inspect(0, 0)[0]).max()
    for m in (60, 80, 87, 95):
        Ro = dom.solve_order(coef, om, tau, m, mu, alpha)
        R, _ = s.plan.inspect(0, m)
        assert np.abs(R - Ro).max() < 1e-9 * top, m
