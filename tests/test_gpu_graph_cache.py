"""The cache of launch graphs: more graphs than it holds, graphs nobody uses any
more beside buffers that change, and replays after an eviction.
"""
import os

import numpy as np
import pytest

import workloads as W
from test_gpu_graph_rule import _direct_us, _host_us
from test_gpu_leafspec import _dev, _same_bits, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

N, LEAF = 300, 100  # 17 launches


def _direct(S, a):
    os.environ["SPIN_NO_GRAPH"] = "1"
    try:
        return S.invert(a, leaf=LEAF).cpu().numpy()
    finally:
        del os.environ["SPIN_NO_GRAPH"]


def test_more_graphs_than_the_cache_holds(torch_cuda):  # noqa: F811
    """80 outputs, each called three times in a row (launched, captured, replayed)
    on other contents each time, then some of the evicted ones again."""
    import paper_1801_04723_amd as S
    torch = torch_cuda
    a = torch.empty(N, N, dtype=torch.float64, device="cuda").t()
    mats = [_dev(torch, W.diag_dominant(N, seed=s)) for s in range(4)]
    want = [_direct(S, m) for m in mats]
    outs = [torch.empty_like(a) for _ in range(80)]
    for i, x in enumerate([*outs, *outs[:6], *outs[40:46]]):
        for r in range(4):
            j = (i + r) % 4
            a.copy_(mats[j])
            x.fill_(float("nan"))
            S.invert(a, leaf=LEAF, out=x)
            (a @ a).sum().item()  # other work and a wait between the calls
            assert _same_bits(x.cpu().numpy(), want[j]), (i, r)
    assert S.info() == 0


def test_unused_graphs_do_not_keep_new_ones_out(torch_cuda):  # noqa: F811
    """63 graphs of buffers not used any more, then two sets in turn."""
    import paper_1801_04723_amd as S
    torch = torch_cuda
    S.release()
    a = _dev(torch, W.diag_dominant(N, seed=1))
    outs = [torch.empty_like(a) for _ in range(65)]
    for x in outs[:63]:
        for _ in range(2):
            S.invert(a, leaf=LEAF, out=x)
    turn = [0]

    def fn():
        turn[0] ^= 1
        S.invert(a, leaf=LEAF, out=outs[63 + turn[0]])

    fn()
    fn()
    assert _host_us(torch, fn) <= 0.75 * _direct_us(torch, fn)


def test_a_third_call_is_replayed(torch_cuda):  # noqa: F811
    """Every kind of call: the third and fourth call equal the direct one, on
    other contents than the captured call's."""
    import paper_1801_04723_amd as S
    torch = torch_cuda
    calls = {"invert": S.invert, "spd": S.invert_spd, "lu": S.invert_lu,
             "mixed": lambda m, leaf, out: S.invert_mixed(m, leaf=leaf, mode="fp32", ns_steps=1, out=out),
             "int8": lambda m, leaf, out: S.invert_mixed(m, leaf=leaf, mode="bf16x3_int8", ns_steps=1, out=out)}
    for kind, f in calls.items():
        a = torch.empty(768, 768, dtype=torch.float64, device="cuda").t()
        x = torch.empty_like(a)
        for r in range(4):
            a.copy_(_dev(torch, W.spd_gram(768, seed=r)))
            x.fill_(float("nan"))
            f(a, leaf=128, out=x)
            (a @ a).sum().item()
            got = x.cpu().numpy()
            y = torch.empty_like(a)
            os.environ["SPIN_NO_GRAPH"] = "1"
            try:
                f(a, leaf=128, out=y)
            finally:
                del os.environ["SPIN_NO_GRAPH"]
            assert np.isfinite(got).all() and _same_bits(got, y.cpu().numpy()), (kind, r)
