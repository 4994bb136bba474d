"""Repeated calls with the same buffers: launched directly at first, captured
on the second call, replayed from then on.  Every call must see the current
contents of its buffers and give the directly launched result, with other GPU
work and waits between the calls."""
import os

import numpy as np
import pytest

import workloads as W
from test_gpu_leafspec import _dev, _same_bits, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

CALLS = {
    "invert": lambda S, a, x, leaf: S.invert(a, leaf=leaf, out=x),
    "spd": lambda S, a, x, leaf: S.invert_spd(a, leaf=leaf, out=x),
    "lu": lambda S, a, x, leaf: S.invert_lu(a, leaf=leaf, out=x),
    "mixed": lambda S, a, x, leaf: S.invert_mixed(a, leaf=leaf, mode="fp32", ns_steps=1, out=x),
}


@pytest.mark.parametrize("kind", sorted(CALLS))
@pytest.mark.parametrize("n,leaf", [(64, 64), (96, 48), (200, 50), (384, 64)])
def test_calls_in_a_row_on_the_same_buffers(torch_cuda, kind, n, leaf):  # noqa: F811
    import paper_1801_04723_amd as S
    torch = torch_cuda
    fn = CALLS[kind]
    a, x = _dev(torch, np.zeros((n, n))), None
    x = torch.empty_like(a)
    for r in range(5):
        m = W.spd_gram(n, seed=100 + r)
        a.copy_(_dev(torch, m))
        x.fill_(float("nan"))
        fn(S, a, x, leaf)
        (a @ a).sum().item()  # other work and a wait between the calls
        got = x.cpu().numpy()
        assert S.info() == 0
        os.environ["SPIN_NO_GRAPH"] = "1"
        try:
            y = torch.empty_like(a)
            fn(S, a, y, leaf)
            want = y.cpu().numpy()
        finally:
            del os.environ["SPIN_NO_GRAPH"]
        assert _same_bits(got, want), r
