"""Pair sums of mutual drop pairs (both directions from one pass over the pairs).

Systems of well-separated drops take the mutual kernel when the viscosity
ratios differ from 1 and the items fill the device; with a ratio of 1 in every
pair the same single layer goes through the direct pair kernel instead, so the
two are compared with each other, and both with the oracle at a sample of
targets. Degrees give target blocks of one and several wavefronts' worth of 64
(N = 144, 180, 544, 612, 1200, 2244 nodes: remainders of 64 targets and of 16
sources, one and three blocks), equal and unequal in a pair.

Tolerance: 1e-10 of the largest value of a component against the oracle (the
FP64 parity bar); 1e-12 between the two kernels (sums of up to 4e4 terms whose
1/r^5 carries at most 5e-14 each, differently grouped).
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


def system(degrees, seed):
    """One drop per degree on a lattice of spacing 6 (region 0 of each other at these degrees)."""
    rng = np.random.default_rng(seed)
    side = int(np.ceil(len(degrees) ** (1 / 3) - 1e-9))
    xs = [W.perturbed_sphere(rng, p, rng.uniform(0.8, 1.2), 6.0 * np.array([k % side, k // side % side, k // side // side]), 0.05)
          for k, p in enumerate(degrees)]
    fs = [W.perturbation(rng, p, 1.0, lmin=1, power=1.5) for p in degrees]
    return xs, fs


def items(degrees, R=256):
    """Items of the mutual plan at runs of R sources: blocks of 1024 targets x runs, over pairs i < j."""
    n = [2 * p * (p + 1) for p in degrees]
    return sum(-(-n[i] // 1024) * -(-n[j] // R) for i in range(len(n)) for j in range(i + 1, len(n)))


CASES = [[16] * 26, [8, 16, 9, 17, 24] * 6, [33, 24, 8] * 4 + [33] * 3]


@pytest.mark.parametrize("degrees", CASES, ids=["p16", "mixed", "large"])
def test_mutual_pairs_match_direct_and_oracle(B, degrees):
    import oracle
    assert items(degrees) >= 3 * 256
    xs, fs = system(degrees, 7)
    nd = len(degrees)
    opts = dict(A_tilde=5.0, U_tilde=2)
    out = {}
    for name, lam in (("mutual", 2.0), ("direct", 1.0)):
        c = B.Context(**opts)
        c.set_drops(degrees, xs, [lam] * nd)
        reg, _ = c.regions()
        assert set(np.unique(reg)) <= {-1, 0}
        out[name] = c.single_layer(fs)
        again = c.single_layer(fs)
        assert all(np.array_equal(a, b) for a, b in zip(out[name], again))
        if name == "mutual":
            dl = c.double_layer(fs, mode=0)
            op = c.double_layer(fs, mode=1)
            # the no-allocation entry point takes the same sums
            import torch
            u = torch.tensor(B.pack_coefficients(fs), device="cuda")
            o = torch.zeros(3 * c.ncoef_total(), dtype=torch.float64, device="cuda")
            B.bim_apply_double_layer_noalloc(c.h, u, o, 1)
            B.bim_synchronize(c.h)
            assert np.array_equal(o.cpu().numpy(), B.pack_coefficients(op))
        c.close()
    for a, b in zip(out["mutual"], out["direct"]):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    s = oracle.System([oracle.Drop(p, x, 2.0, None, f) for p, x, f in zip(degrees, xs, fs)], oracle.Options(**opts))
    for i in (0, 1, nd // 2, nd - 1):
        n = oracle.npts(degrees[i])
        tg = np.array([0, 63, 64, n // 2, n - 1])
        for got, kind, scale in ((out["mutual"][i], 0, -8 * np.pi), (dl[i], 1, 4 * np.pi)):
            ref = s.layer(i, fs, kind, targets=tg)
            err = max(np.abs(got[tg, k] * scale - ref[:, k]).max() / np.abs(ref[:, k]).max() for k in range(3))
            assert err <= 1e-10, (i, kind, err)
