"""Stand-alone FP64 transforms: which field counts take the matrix cores, and the
matrix cores against the oracle at sizes where few fields no longer take them.

The line: 24 fields, and 1600 synthesis blocks (fields x latitude pairs x runs of
64 longitudes) up to degree 61, 1110 above. A field's bits do not depend on how
many others are transformed with it by the same kernels, and differ between the two
forms, so they show which one ran.

Tolerance against the oracle: 1e-10 of a field's largest value (synthesis) or
coefficient (analysis), the FP64 bar of the transforms.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


def coefficients(p, nf, seed):
    c = np.random.default_rng(seed).standard_normal((nf, (p + 1) * (p + 2) // 2, 2))
    c[:, [n * (n + 1) // 2 for n in range(p + 1)], 1] = 0.0
    return c


def synthesis(B, c, p, q, coef):
    g = np.zeros(len(coef) * B.npts(q))
    B.bim_sh_synthesize(c.h, p, q, len(coef), np.ascontiguousarray(coef.reshape(-1)), 0, 0, g)
    return g.reshape(len(coef), -1)


# (degree, grid, most fields that take the batched form)
LINE = [(16, 16, 24), (61, 127, 24), (30, 128, 12), (61, 128, 12), (62, 90, 24), (62, 128, 8), (63, 100, 21), (63, 126, 17),
        (63, 128, 8)]


@pytest.mark.parametrize("p,q,most", LINE)
def test_field_count_line(B, p, q, most):
    coef = coefficients(p, 25, 10 * p + q)
    c = B.Context()
    cores = synthesis(B, c, p, q, coef)
    few, more = synthesis(B, c, p, q, coef[:most]), synthesis(B, c, p, q, coef[:most + 1])
    c.close()
    assert np.array_equal(more, cores[:most + 1])
    assert not np.array_equal(few, cores[:most])
    assert np.abs(few - cores[:most]).max() <= 1e-10 * np.abs(cores).max()


@pytest.mark.parametrize("p,q", [(13, 39), (31, 62), (40, 120), (63, 63), (63, 126)])
def test_matrix_core_synthesis(B, orc, p, q):
    coef = coefficients(p, 25, 20 * p + q)
    c = B.Context()
    g = synthesis(B, c, p, q, coef)
    c.close()
    for f in range(25):
        ref = orc.synth(p, coef[f], q, 0, 0).ravel()
        assert np.abs(g[f] - ref).max() <= 1e-10 * np.abs(ref).max()


@pytest.mark.parametrize("q,p", [(17, 17), (33, 20), (45, 30), (63, 63)])
def test_matrix_core_analysis(B, orc, q, p):
    g = np.random.default_rng(30 * p + q).standard_normal((25, B.npts(q)))
    c = B.Context()
    out = np.zeros(25 * 2 * B.ncoef(p))
    B.bim_sh_analyze(c.h, q, p, 25, np.ascontiguousarray(g.reshape(-1)), out)
    few = np.zeros(2 * B.ncoef(p))
    B.bim_sh_analyze(c.h, q, p, 1, np.ascontiguousarray(g[0]), few)
    c.close()
    out = out.reshape(25, -1, 2)
    assert not np.array_equal(out[0].reshape(-1), few)  # the two forms' last bits differ
    for f in range(25):
        ref = orc.analyze(g[f], q, p)
        assert np.abs(out[f] - ref).max() <= 1e-10 * np.abs(ref).max()
