"""Uniform tension reads no surfactant fields: what an earlier equation of state
left in the work buffer (here values that overflow) does not reach the force."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_uniform_force_after_an_overflowing_surfactant():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    p = 8
    x = W.perturbed_sphere(np.random.default_rng(1), p, 1.0, (0, 0, 0), 0.05)
    a = B.Context()
    a.set_drops([p], [x], [1.0])
    want = a.force()[0]
    g = np.full((B.ncoef(p), 2), 1e308)  # finite coefficients, infinite values on the grid
    a.set_tension([g], B.BIM_EOS_LINEAR, E=0.5, xs=0.6)
    a.force()
    a.set_tension(None, B.BIM_EOS_UNIFORM)
    assert np.array_equal(a.force()[0], want) and np.all(np.isfinite(want))
    a.close()
