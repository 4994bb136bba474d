"""Whole leaves with the diagonal chain one block step ahead.

Half of the panels' updates run on the matrix cores with zeros for the steps
that a value does not take, which must leave every bit (signed zeros too) as
the search computes it; where a value on the way is not finite the leaf goes to
the search.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_leafblocks import _compare
from test_gpu_leafspec import _same_bits, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

ORDERS = (17, 48, 64, 65, 96, 97, 128)


@pytest.mark.parametrize("L", ORDERS)
@pytest.mark.parametrize("shape", ["lower", "upper", "arrow", "blocks"])
def test_exact_zeros_keep_their_signs(torch_cuda, L, shape):  # noqa: F811
    A = W.diag_dominant(L, seed=L)
    i, j = np.indices(A.shape)
    keep = {"lower": j <= i, "upper": j >= i, "arrow": (i == j) | (i == L - 1) | (j == 0),
            "blocks": (i // 7) == (j // 7)}[shape]
    A[~keep] = 0.0
    A[(~keep) & ((i + j) % 3 == 0)] = -0.0
    A[::2] *= -1.0
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st == 0 and _same_bits(x0, x1)


@pytest.mark.parametrize("L", ORDERS)
@pytest.mark.parametrize("at", ["first", "middle", "last"])
def test_overflow_goes_to_the_search(torch_cuda, L, at):  # noqa: F811
    # row k of U overflows when it is divided by its pivot
    k = {"first": 0, "middle": L // 2, "last": L - 2}[at]
    A = np.eye(L)
    A[k, k] = 2.0 ** -490
    A[k, L - 1] = 2.0 ** 700
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st != 0 or _same_bits(x0, x1)


@pytest.mark.parametrize("L", [63, 100, 128])
def test_offset_and_padded_operands(torch_cuda, L):  # noqa: F811
    torch = torch_cuda
    import paper_1801_04723_amd as S
    from test_gpu_leafspec import _both
    buf = torch.zeros(L + 5, L + 3, dtype=torch.float64, device="cuda")
    A = buf[2:L + 2, 1:L + 1]
    A.copy_(torch.from_numpy(W.diag_dominant(L, seed=L)))
    for a in (A, A.t()):
        x0, s0, x1, s1 = _both(lambda: S.invert(a, leaf=L))
        assert s0 == s1 == 0 and _same_bits(x0, x1)
