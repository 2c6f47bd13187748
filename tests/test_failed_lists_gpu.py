"""Pair work lists that cannot be built are not taken for built ones by the next
call: 2400 drops of degree 2 have 5.8e6 pairs of drops, one work item each, whose
partial sums pass what a slot index can address (3 x 128 doubles an item), so the
single layer is refused after the regions are there, each time it is called. The
same context then evaluates drops that fit as a new one does.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_refused_lists_stay_refused():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    p, nd = 2, 2400
    rng = np.random.default_rng(2)
    few = [W.perturbed_sphere(rng, p, 1.0, (4.0 * k, 0, 0), 0.0) for k in range(3)]
    fs = [W.perturbation(rng, p, 1.0, lmin=1, power=1.5) for _ in few]
    c = B.Context(U_tilde=1, U_geom=1, pair_tune=0)
    c.set_drops([p] * 3, few, [1.0] * 3)
    want = c.single_layer(fs)
    xs = [few[0].copy() for _ in range(nd)]
    for k, x in enumerate(xs):  # a lattice of spacing 6, drops in each other's region 0
        x[:, 0, 0] += np.sqrt(4 * np.pi) * 6.0 * np.array([k % 14, k // 14 % 14, k // 196])
    c.set_drops([p] * nd, xs, [1.0] * nd)
    f, out = np.zeros(3 * nd * 2 * B.ncoef(p)), np.zeros(3 * nd * B.npts(p))
    for _ in range(2):
        with pytest.raises(B.BimError) as e:
            B.bim_single_layer(c.h, f, out)
        assert e.value.status == B.BIM_ENOMEM, e.value
    c.set_drops([p] * 3, few, [1.0] * 3)
    assert all(np.array_equal(a, b) for a, b in zip(c.single_layer(fs), want))
    c.close()
