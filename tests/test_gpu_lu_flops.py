"""Traced operations of the LU schedule's launches: without the zero triangles
that its products skip, so that traced rates are rates of work done."""
import pytest

import oracle
from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _lu_flops(m, leaf):
    """Direct sum over the recursion: 4/3 L^3 per leaf; per node S (2 n2 n2 n1)
    and six products with a triangle of order h, each of whose entries meets half
    of the other operand: h (h + 1) times the other side."""
    if m <= leaf:
        return 4.0 / 3.0 * m ** 3
    n1 = oracle.split(m)
    n2 = m - n1
    # U12, L21, T1, T2 with triangles of order n1; Li21, Ui12 with order n2
    return (_lu_flops(n1, leaf) + _lu_flops(n2, leaf) + 2 * n2 * n2 * n1
            + 4 * n1 * (n1 + 1) * n2 + 2 * n2 * (n2 + 1) * n1)


@pytest.mark.parametrize("n,leaf", [(1, 1), (129, 64), (300, 64), (640, 128), (2048, 128)])
def test_traced_flops(torch_cuda, n, leaf):  # noqa: F811
    import paper_1801_04723_amd as S
    import workloads as W
    a = W.torch_diag_dominant(n, 3)
    S.trace_enable(True)
    try:
        S.invert_lu(a, leaf=leaf)
        torch_cuda.cuda.synchronize()
        recs = S.trace_collect()
    finally:
        S.trace_enable(False)
    # X = Ui Li: entry (i, j) sums k = max(i, j) .. n - 1
    last = sum(2 * (2 * s + 1) * (n - s) for s in range(n))
    assert sum(r["flops"] for r in recs) == pytest.approx(_lu_flops(n, leaf) + last, rel=1e-12)
