"""The fast summation's kernels over the orders where their launches change:
one to eight wavefronts of coefficients (order 9 is the last with one, 30 the
largest), both layers, against direct sums.

Two spheres of radius 1 at distance D: rho = 2 / D, and fmm_eps = 3 rho^(P+1)
lets the pair take order P and no lower one. Tolerance: the truncated series
of 1/r in the two radii starts at rho^(P+1) times 1/D; a velocity takes up to
two derivatives of it, each at most a factor P + 2 on the radius 1, so the
difference stays below 4 (P + 2)^2 rho^(P+1) of the largest direct value,
plus 1e-12 for the rounding of the sums.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.mark.parametrize("P", [2, 3, 9, 10, 15, 24, 30])
@pytest.mark.parametrize("p", [5, 12])
def test_orders_against_direct(B, P, p):
    D = 5.0
    rho = 2.0 / D
    rng = np.random.default_rng(10 * P + p)
    xs = [W.sphere(p, 1.0, (0.0, 0.0, 0.0)), W.sphere(p, 1.0, (0.6 * D, 0.0, 0.8 * D))]
    u = [W.perturbation(rng, p, 1.0, lmin=1, power=2.0) for _ in xs]
    z = np.zeros_like(u[0])
    got = []
    for order in (0, P):
        c = B.Context(A_tilde=0.5, fmm_order=order, fmm_eps=3.0 * rho ** (P + 1))
        c.set_drops([p, p], xs, [2.0, 3.0])
        # the second drop carries the density: the first one's values are the far field
        got.append((c.single_layer([z, u[1]])[0], c.double_layer([z, u[1]], mode=0)[0]))
        c.close()
    for direct, fast in zip(*got):
        assert np.all(np.isfinite(fast))
        assert not np.array_equal(direct, fast)  # the pair did take the fast summation
        tol = 4.0 * (P + 2) ** 2 * rho ** (P + 1) + 1e-12
        assert np.abs(fast - direct).max() <= tol * np.abs(direct).max(), (P, p)
