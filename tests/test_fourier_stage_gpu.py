"""The Fourier stage of the singular pipeline at the edges of its tiles.

Degrees and singular grids are chosen where the stage changes shape: one and
several depth steps of four even orders (p = 7, 8), row counts qs/2 + 1 at and
past a tile (4, 8, 9, 16, 17, 25, 28 rows; one to four wavefronts), odd qs (no
row at phi = pi/2), a singular grid finer than the degree (U_sing = 2: rows
without orders), target counts that are no multiple of 16, and the largest
degree of the pipeline (51). Single layer, stored double layer and both in one
pass (a solve) against the oracle's pole rule.

Tolerance: the FP64 parity bar of the other parity tests, 1e-10 of the largest
value of a component; the sums here have at most 112 terms and the stresslet's
h.n loses about p^2 eps = 6e-13 at the ring nearest the pole.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-10
CASES = [(2, 1), (3, 1), (5, 2), (7, 1), (8, 1), (9, 1), (14, 1), (15, 1), (15, 2), (16, 1), (17, 1), (25, 2), (31, 1),
         (33, 1), (48, 1), (51, 1)]


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.mark.parametrize("p,us", CASES)
def test_self_layers_against_oracle(B, p, us):
    import oracle
    rng = np.random.default_rng(100 * p + us)
    xc = W.perturbed_sphere(rng, p, 1.0, (0.3, -0.2, 0.1), 0.05)
    f = W.perturbation(rng, p, 1.0, lmin=1, power=1.5)
    # a few targets of every kind: first and last latitude, the middle one, all residues mod 16
    n = oracle.npts(p)
    tg = np.unique(np.concatenate([np.arange(min(n, 3)), n // 2 + np.arange(min(n - n // 2, 17 if p < 40 else 2)), [n - 1]]))
    ref = [oracle.singular(p, xc, f, kind, tg, us * p) for kind in (0, 1)]
    c = B.Context(U_sing=us)
    c.set_drops([p], [xc], [2.0])
    s = c.single_layer([f])[0] * (-8.0 * np.pi)
    d = c.double_layer([f], mode=0)[0] * (4.0 * np.pi)
    for got, want in ((s, ref[0]), (d, ref[1])):
        assert np.all(np.isfinite(got))
        err = max(np.abs(got[tg, k] - want[:, k]).max() / np.abs(want[:, k]).max() for k in range(3))
        assert err <= TOL, (p, us, err)
    # both layers in one pass: the operator's rows built with the single layer
    # equal those built alone
    e = B.Context(U_sing=us)
    e.set_drops([p], [xc], [2.0])
    e.eval_velocity(coefficients=True)
    d2 = e.double_layer([f], mode=0)[0] * (4.0 * np.pi)
    assert np.abs(d2 - d).max() <= 1e-13 * np.abs(d).max()
    c.close()
    e.close()
