"""Stand-alone transforms of few fields against many: up to 24 fields (grids to
degree 128) take one batched launch, more the matrix cores, and a field's result
is the same within rounding, on host and on device memory, on both sides of
the line.

Tolerance: both forms add the same terms in another order. Synthesis: (p + 1)
(p + 2)/2 terms per value, in nested sums of at most p + 1 each, magnitudes A = 2
sum |c_nm| sqrt(n + 1/2): below 4 (p + 1) eps A apart, 16 with the recurrences of
the phases. Analysis: 2q longitudes and q + 1 latitudes with weights that add up to
4 pi: below 16 (3q + 1) eps 4 pi sqrt(p + 1/2) max |v|.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps
SIZES = [(0, 1), (5, 5), (16, 16), (16, 33), (31, 31), (48, 48), (63, 63), (20, 128), (20, 129)]


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.mark.parametrize("p,q", SIZES)
def test_few_fields_equal_many(B, p, q):
    import torch
    rng = np.random.default_rng(100 * p + q)
    nc, nq, nf = (p + 1) * (p + 2) // 2, 2 * q * (q + 1), 25
    n = np.repeat(np.arange(p + 1), np.arange(1, p + 2))
    coef = rng.standard_normal((nf, nc, 2))
    coef[:, [k * (k + 1) // 2 for k in range(p + 1)], 1] = 0.0
    c = B.Context()

    def both(k):
        g, a = np.zeros(k * nq), np.zeros(k * 2 * nc)
        B.bim_sh_synthesize(c.h, p, q, k, np.ascontiguousarray(coef[:k].reshape(-1)), 0, 0, g)
        B.bim_sh_analyze(c.h, q, p, k, g, a)
        return g.reshape(k, nq), a.reshape(k, nc, 2)

    g0, a0 = both(nf)
    A = 2.0 * (np.abs(coef).sum(axis=2) * np.sqrt(n + 0.5)).sum(axis=1)
    for k in (1, 3, 4, 24):
        g, a = both(k)
        assert np.all(np.abs(g - g0[:k]).max(axis=1) <= 16 * (p + 1) * EPS * A[:k])
        # the analyses read values that differ by the bound above
        bound = (16 * (3 * q + 1) * EPS * np.abs(g).max(axis=1) + 16 * (p + 1) * EPS * A[:k]) * 4 * np.pi * np.sqrt(p + 0.5)
        assert np.all(np.abs(a - a0[:k]).max(axis=(1, 2)) <= bound)
    # device memory: the same bits as through the host
    d = torch.from_numpy(coef[:3].reshape(-1).copy()).cuda()
    out = torch.zeros(3 * nq, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    B.bim_sh_synthesize(c.h, p, q, 3, d, 0, 0, out)
    B.bim_synchronize(c.h)
    assert np.array_equal(out.cpu().numpy(), both(3)[0].reshape(-1))
    c.close()
