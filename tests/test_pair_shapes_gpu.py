"""The timed work shape of the direct pair sums (option pair_tune) belongs to the
pairs it was timed on.

Fourteen drops of degree 40, two of them close to each other: in FP64 all pairs
but that one take the mutual kernel, so the shape is for a hundredth of the
2.0e9 pairs that a mixed-precision context of the same drops sums directly.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

P, ND = 40, 14


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.fixture(scope="module")
def drops():
    rng = np.random.default_rng(40)
    at = [6.0 * np.array([k % 3, k // 3 % 3, k // 9]) for k in range(ND)]
    at[-1] = at[0] + np.array([2.2, 0.0, 0.0])
    xs = [W.perturbed_sphere(rng, P, 1.0, c, 0.02) for c in at]
    fs = [W.perturbation(rng, P, 1.0, lmin=1, power=1.5) for _ in at]
    return xs, fs


OPTS = dict(A_tilde=5.0, U_tilde=2)


def test_shape_of_one_precision_is_not_taken_for_the_other(B, drops):
    """FP64 first, then mixed: the mixed context's partial sums fit the
    no-allocation scratch, as they do by the rule (576 sources an item: 10e6
    doubles), and both entry points give the same bits."""
    import torch
    xs, fs = drops
    c = B.Context(**OPTS)
    c.set_drops([P] * ND, xs, [2.0] * ND)
    c.single_layer(fs)
    assert 1 in c.regions()[0]  # pairs are left for the direct kernel
    c.close()
    c = B.Context(precision=B.BIM_PREC_MIXED, **OPTS)
    c.set_drops([P] * ND, xs, [2.0] * ND)
    want = B.pack_coefficients(c.double_layer(fs, mode=1))
    u = torch.tensor(B.pack_coefficients(fs), device="cuda")
    out = torch.zeros(len(want), dtype=torch.float64, device="cuda")
    rc = B.lib().bim_apply_double_layer_noalloc(c.h, u.data_ptr(), out.data_ptr(), 1)
    assert rc == B.BIM_OK, B.lib().bim_last_error(c.h)
    B.bim_synchronize(c.h)
    assert np.array_equal(out.cpu().numpy(), want)
    c.close()


def test_only_the_direct_pairs_are_timed(B, drops):
    """The timed passes leave out what no candidate changes: all of them together
    (double layers; the call itself is a single layer) count fewer pairs than one
    pass over the mutual ones (41e6 direct pairs, 21 passes at most, 1.7e9)."""
    keep = [0] + list(range(2, ND))  # a drop less, the close pair in: a shape that is not stored yet
    xs, fs = ([v[k] for k in keep] for v in drops)
    nd = len(keep)
    c = B.Context(**OPTS)
    c.set_drops([P] * nd, xs, [2.0] * nd)
    B.bim_profile(c.h, 1)
    c.single_layer(fs)
    timed = B.bim_profile_query(c.h, "pair_dl")
    c.close()
    mutual = (nd * (nd - 1) / 2 - 1) * 2.0 * B.npts(P) ** 2
    assert timed["launches"] > 0
    assert timed["flops"] < 30.0 * mutual, (timed, 30.0 * mutual)
