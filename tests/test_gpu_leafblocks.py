"""Leaves eliminated 16 steps at a time on the matrix cores.

The speculative elimination of a leaf runs in blocks of 16 steps (one serial
chain per diagonal block, the rest as matrix-core updates), with the operations
of the pivot search in the same order, so its result is the search's bit for
bit: at every order around the 16- and 64-wide blocks, with a failing check in
any block, and for values at the edges of the format.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_leafspec import _both, _dev, _same_bits, _swap_rows, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = (2, 15, 16, 17, 31, 32, 33, 47, 48, 63, 65, 80, 111, 112, 113, 127, 257, 272, 319, 321, 449, 511)


def _compare(torch, A, L):
    import paper_1801_04723_amd as S
    dA = _dev(torch, A)
    x0, s0, x1, s1 = _both(lambda: S.invert(dA, leaf=L))
    assert s0 == s1
    return x0, x1, s1


@pytest.mark.parametrize("L", EDGES)
def test_block_edges_equal_search(torch_cuda, L):  # noqa: F811
    x0, x1, st = _compare(torch_cuda, W.diag_dominant(L, seed=3 * L), L)
    assert st == 0 and _same_bits(x0, x1)
    # row-major input and an FP32 leaf (mixed mode, no refinement)
    import paper_1801_04723_amd as S
    torch = torch_cuda
    a = torch.from_numpy(np.ascontiguousarray(W.diag_dominant(L, seed=5 * L))).cuda()
    x0, s0, x1, s1 = _both(lambda: S.invert_mixed(a, leaf=L, mode="fp32", ns_steps=0))
    assert s0 == s1 == 0 and _same_bits(x0, x1)


@pytest.mark.parametrize("L,step", [(64, 0), (64, 15), (64, 16), (100, 47), (100, 98), (128, 16), (128, 95),
                                    (128, 111), (300, 63), (300, 64), (300, 260), (512, 447)])
def test_failed_check_in_any_block(torch_cuda, L, step):  # noqa: F811
    A = _swap_rows(W.diag_dominant(L, seed=L + step), step, step + 1)
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st == 0 and _same_bits(x0, x1)


@pytest.mark.parametrize("L", [20, 64, 128, 320])
@pytest.mark.parametrize("scale", [-600, -499, 499, 600])
def test_pivots_outside_the_plain_range(torch_cuda, L, scale):  # noqa: F811
    A = np.ldexp(W.diag_dominant(L, seed=L), scale)
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st == 0 and _same_bits(x0, x1)


@pytest.mark.parametrize("L", [33, 64, 128, 300])
def test_signed_zeros_and_non_finite(torch_cuda, L):  # noqa: F811
    A = W.diag_dominant(L, seed=9)
    A[L // 2:, : L // 2] = -0.0
    A[: L // 2, L // 2:] = 0.0
    x0, x1, st = _compare(torch_cuda, A, L)
    assert st == 0 and _same_bits(x0, x1)
    for bad in (np.inf, np.nan):
        B = W.diag_dominant(L, seed=10)
        B[L - 3, L - 9] = bad
        _, _, st = _compare(torch_cuda, B, L)
        assert st > 0
