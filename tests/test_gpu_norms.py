"""Frobenius norms and the refinement's grouped auxiliary launches: the residual
measure at orders around the kernel's waves and blocks, from repeated calls on
one workspace, and a batch of more mixed requests than one grouped launch holds,
each equal to its solo result bit for bit."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_leafspec import _dev, _same_bits, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 129, 255, 257, 700, 1025])
def test_residual_measure(torch_cuda, n):  # noqa: F811
    import paper_1801_04723_amd as S
    g = np.random.default_rng(n)
    A, X = g.standard_normal((n, n)), g.standard_normal((n, n))
    want = oracle.residual(A, X)
    dA, dX = _dev(torch_cuda, A), _dev(torch_cuda, X)
    got = [S.residual(dA, dX) for _ in range(3)]
    assert got[0] == got[1] == got[2]  # fixed summation order
    # squares summed in any order: n^2 terms, and the product's rounding
    assert abs(got[0] - want) <= 4 * (n + 2) * 2.0 ** -53 * np.sqrt(n) * want


def test_more_requests_than_a_grouped_launch(torch_cuda):  # noqa: F811
    import paper_1801_04723_amd as S
    torch = torch_cuda
    orders = [64 + 8 * (i % 9) for i in range(70)]
    mats = [_dev(torch, W.spd_gram(n, seed=i)) for i, n in enumerate(orders)]
    outs, info = S.invert_batch(mats, leaf=64, modes=["fp32"] * 70, ns_steps=2)
    assert info == [0] * 70
    for a, x in zip(mats, outs):
        y = S.invert_mixed(a, leaf=64, mode="fp32", ns_steps=2)
        assert _same_bits(x.cpu().numpy(), y.cpu().numpy())
