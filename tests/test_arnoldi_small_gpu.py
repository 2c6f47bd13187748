"""Arnoldi steps by one block and by three kernels: solves on both sides of the
rule's edges.

Sizes n = 3 (p+1)(p+2) per drop: the smallest (p = 2, n = 36), fewer entries
than one wavefront pass, a size that stays with the one-block form throughout,
one that leaves it after ten vectors, one just below 8192 entries and one just
above it; restarts short enough that the basis starts again inside a solve.

The solution u satisfies A u = b with the operator and the right-hand side
formed by the other entry points (b = P[2 x single layer] without far field),
to the requested 1e-12 plus the rounding of the operator (1e-14 per term, n
terms at most in a sum: 1e-10 / 1e3); checked at 1e-11 ||b||.
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


@pytest.mark.parametrize("p,nd,restart", [(2, 1, 50), (4, 1, 3), (16, 2, 50), (16, 2, 5), (35, 2, 50), (35, 2, 4), (36, 2, 50),
                                          (36, 2, 4)])
def test_solution_satisfies_the_equation(B, p, nd, restart):
    rng = np.random.default_rng(10 * p + nd)
    xs = [W.perturbed_sphere(rng, p, 1.0, (3.0 * k, 0.2, 0.0), 0.05) for k in range(nd)]
    c = B.Context(gmres_tol=1e-12, gmres_restart=restart, gmres_maxit=400, U_tilde=2)
    c.set_drops([p] * nd, xs, [5.0, 3.0][:nd])
    u, rep = c.eval_velocity(coefficients=True)
    assert rep.gmres_iterations > 0 and rep.gmres_residual <= 1e-12
    au = c.double_layer(u, mode=1)
    s = c.single_layer()
    num = den = 0.0
    for k in range(nd):
        g = np.ascontiguousarray(2.0 * s[k].T)
        b = np.zeros((3, B.ncoef(p), 2))
        B.bim_sh_analyze(c.h, p, p, 3, g, b)
        num += ((au[k] - b) ** 2).sum()
        den += (b ** 2).sum()
    assert np.sqrt(num / den) <= 1e-11, (p, nd, restart, np.sqrt(num / den), rep.gmres_iterations)
    again = c.eval_velocity(coefficients=True)[0]
    assert all(np.array_equal(a, b) for a, b in zip(u, again))
    c.close()
