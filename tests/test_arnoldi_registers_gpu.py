"""Arnoldi steps with the basis in registers, at the edges of their sizes and
vector counts: n = 6 (p + 1)(p + 2)/2 per drop just above 2048 (p = 17), inside and
just below 4096 (p = 21, 24), just above it (p = 25), and restarts at, below and
above the most vectors each size keeps (16, 9, 4), so that a solve passes
from one form to the next. The check and its tolerance are those of the
one-block form's test.
"""
import pytest

import test_arnoldi_small_gpu as base

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_02156_amd as B
    return B


@pytest.mark.parametrize("p,nd,restart", [(3, 1, 16), (16, 2, 16), (16, 2, 17), (17, 2, 9), (17, 2, 50), (21, 2, 10), (24, 2, 50),
                                          (25, 2, 4), (25, 2, 50)])
def test_solution_satisfies_the_equation(B, p, nd, restart):
    base.test_solution_satisfies_the_equation(B, p, nd, restart)
