"""The no-allocation operator on drops without pairs (one drop; drops of different
systems): a mode that has not been applied is refused, as with pairs, and works
once bim_apply_double_layer or a velocity evaluation has applied it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd", [1, 2], ids=["one drop", "two systems"])
def test_mode_not_applied_is_refused(nd):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    p = 8
    rng = np.random.default_rng(9)
    xs = [W.perturbed_sphere(rng, p, 1.0, (0.5 * k, 0, 0), 0.05) for k in range(nd)]
    us = [W.perturbation(rng, p, 1.0, lmin=1, power=1.5) for _ in xs]
    c = B.Context()
    u = torch.tensor(B.pack_coefficients(us), dtype=torch.float64, device="cuda")
    n = [3 * nd * B.npts(p), 3 * nd * 2 * B.ncoef(p)]

    def noalloc(mode):
        out = torch.zeros(n[mode], dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        rc = B.lib().bim_apply_double_layer_noalloc(c.h, u.data_ptr(), out.data_ptr(), mode)
        B.bim_synchronize(c.h)
        return rc, out.cpu().numpy()

    def drops():
        c.set_drops([p] * nd, xs, [3.0, 5.0][:nd])
        if nd > 1:
            c.set_systems(list(range(nd)))

    drops()
    assert noalloc(0)[0] == noalloc(1)[0] == B.BIM_ESTATE  # nothing is built
    for first in (0, 1):
        drops()
        c.double_layer(us, mode=first)
        assert noalloc(1 - first)[0] == B.BIM_ESTATE, first
        want = B.pack_coefficients(c.double_layer(us, mode=1))
        rc, got = noalloc(1)
        assert rc == B.BIM_OK, B.lib().bim_last_error(c.h)
        assert np.array_equal(got, want)
    # a velocity evaluation applies mode 1
    drops()
    c.set_tension(None, 0, sigma0=1.0)
    c.eval_velocity()
    assert noalloc(0)[0] == B.BIM_ESTATE
    rc, got = noalloc(1)
    assert rc == B.BIM_OK and np.array_equal(got, want)
    c.close()
