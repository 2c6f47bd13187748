"""bim_set_drops that fails after its arguments were accepted (here: upsampled
nodes of 756 GB, more than the device has) leaves a context with no drops: no
sizes of the new drops beside the tables of the old ones. The next set of drops
works as on a new context. An argument that is refused leaves the old drops.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

P = 8


def test_failed_allocation_leaves_no_drops():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    rng = np.random.default_rng(8)
    xs = [W.perturbed_sphere(rng, P, 1.0, c, 0.05) for c in ((0, 0, 0), (2.6, 0, 0))]
    fs = [W.perturbation(rng, P, 1.0, lmin=1, power=1.5) for _ in xs]
    c = B.Context(U_tilde=64)
    c.set_drops([P] * 2, xs, [1.0, 5.0])
    want = c.single_layer(fs)
    with pytest.raises(B.BimError) as e:
        c.set_drops([P, 65], xs, [1.0, 5.0])
    assert e.value.status == B.BIM_EINVAL
    c.ps = [P] * 2
    assert all(np.array_equal(a, b) for a, b in zip(c.single_layer(fs), want))
    nd = 60000
    with pytest.raises(B.BimError) as e:
        B.bim_set_drops(c.h, [P] * nd, np.tile(xs[0].reshape(3, 1, -1), (1, nd, 1)).reshape(-1), [1.0] * nd)
    assert e.value.status == B.BIM_ENOMEM, e.value
    out = np.zeros(3 * 2 * B.npts(P))
    for call in (lambda: B.bim_single_layer(c.h, B.pack_coefficients(fs), out), lambda: c.eval_velocity(),
                 lambda: c.set_systems([0, 1])):
        with pytest.raises(B.BimError) as e:
            call()
        assert e.value.status == B.BIM_ESTATE
    c.set_drops([P] * 2, xs, [1.0, 5.0])
    assert all(np.array_equal(a, b) for a, b in zip(c.single_layer(fs), want))
    c.close()
