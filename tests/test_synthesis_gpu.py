"""The batched synthesis at its edges: values and every derivative set, degrees
at and past what its LDS holds, odd and even grid degrees (mirrored latitudes
with and without a middle one; longitudes on the symmetry axes), grids finer
than the degree and more than one block of longitudes, and field counts that
leave a job with one, two or three components.

Tolerance: each output is a sum of (p + 1)(p + 2)/2 terms c_nm d^dt(Ptilde) (i m)^dp
e^{i m phi}. The Legendre entries of both sides come from recursions of length n
(relative error below 8 n eps of the largest entry of the degree) and a sum of N
terms adds at most N eps of the sum of their magnitudes, so with A the sum over
n, m of |c_nm| m^dp max_theta |d^dt Ptilde_n^m| the difference stays below
16 (p + 1) eps A.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SETS = [(0, 0), (1, 0), (0, 1), (2, 0), (1, 1), (0, 2)]
SIZES = [(0, 1, 1), (1, 1, 3), (2, 3, 4), (16, 16, 5), (16, 33, 3), (31, 32, 4), (32, 64, 3), (40, 131, 2), (64, 65, 3),
         (101, 101, 1), (121, 130, 2)]


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.mark.parametrize("p,q,nf", SIZES)
def test_synthesis_against_oracle(B, p, q, nf):
    import oracle
    rng = np.random.default_rng(1000 * p + q)
    nc = (p + 1) * (p + 2) // 2
    coef = rng.standard_normal((nf, nc, 2)) / (1.0 + np.arange(nc))[None, :, None] ** 0.5
    n = np.repeat(np.arange(p + 1), np.arange(1, p + 2))
    m = np.concatenate([np.arange(k + 1) for k in range(p + 1)])
    coef[:, m == 0, 1] = 0.0
    c = B.Context()
    for dt, dp in SETS:
        out = np.zeros(nf * (q + 1) * 2 * q)
        B.bim_sh_synthesize(c.h, p, q, nf, np.ascontiguousarray(coef.reshape(-1)), dt, dp, out)
        out = out.reshape(nf, q + 1, 2 * q)
        assert np.all(np.isfinite(out))
        for f in range(nf):
            # |Ptilde| <= sqrt((2n + 1)/2), a derivative brings at most a factor n + 1 (n, m <= n)
            A = 2.0 * np.sum(np.abs(coef[f]).sum(axis=1) * np.sqrt(n + 0.5) * (n + 1.0) ** dt * m ** float(dp))
            ref = oracle.synth(p, coef[f], q, dt, dp)
            assert np.abs(out[f] - ref).max() <= 16 * (p + 1) * np.finfo(float).eps * A, (p, q, f, dt, dp)
    c.close()
