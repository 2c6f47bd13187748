"""Stored double-layer rows in the launch of the density synthesis.

With launches timed one by one the two run apart: the joint launch must give
the same bits (it stores w M u where the other adds it to a cleared value).
Drops of one and of several degrees (jobs of different lengths, tails of the
row blocks), a drop without a double layer (its values are the pair sums
alone), one drop alone, a call that follows another of the same context, and
more drops than one launch holds.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

CASES = [([3], [2.0]), ([16], [5.0]), ([16, 16], [3.0, 1.0]), ([7, 12, 5], [2.0, 1.0, 0.5]), ([32, 9], [1.0, 4.0]),
         ([2] * 35, [2.0] * 35)]


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.mark.parametrize("ps,lam", CASES)
def test_joint_launch_equals_separate_ones(B, ps, lam):
    rng = np.random.default_rng(len(ps) + ps[0])
    xs = [W.perturbed_sphere(rng, p, 1.0, (3.2 * (i % 6), 3.2 * (i // 6), 0.1 * i), 0.02) for i, p in enumerate(ps)]
    us = [W.perturbation(rng, p, 1.0, lmin=1, power=1.5) for p in ps]
    c = B.Context(xform_path=1, pair_tune=0)
    c.set_drops(ps, xs, lam)
    got = []
    for timed in (0, 1, 0):
        B.bim_profile(c.h, timed)
        got.append(c.double_layer(us, mode=0))
    for a, b in ((0, 1), (0, 2)):
        for x, y in zip(got[a], got[b]):
            assert np.all(np.isfinite(x)) and np.array_equal(x, y)
    c.close()
