"""The choice of a product's kernel: across a line of the choice the time grows
with the work.  Each case compares two products of nearly the same size, whose
times may differ by the ratio of their work and one part in twelve."""
import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _us(torch, mode, m, n, k, beta):
    import paper_1801_04723_amd as S
    dt = torch.float64 if mode == "fp64" else torch.float32
    a, b, c = (torch.randn(x, y, dtype=dt, device="cuda") for x, y in ((k, m), (n, k), (n, m)))
    d = torch.empty_like(c)
    best = float("inf")
    for _ in range(8):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(20):
            S.gemm_cm(m, n, k, -1.0, a, m, b, k, beta, c, m, d, m, dtype=mode)
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1) * 50.0)
    return best


@pytest.mark.parametrize("mode,size,less,beta", [
    # plain BF16 below one round of 256 x 256 tiles
    ("bf16", (2048, 5120, 768), (2048, 4864, 768), 0.0),
    # ragged FP32 with a short k, where 128 x 128 tiles need a second round
    ("fp32", (3201, 3201, 100), (2801, 2801, 100), 0.0),
])
def test_time_grows_with_the_work(torch_cuda, mode, size, less, beta):  # noqa: F811
    torch = torch_cuda
    _us(torch, mode, *less, beta)
    work = (size[0] * size[1] * size[2]) / (less[0] * less[1] * less[2])
    assert _us(torch, mode, *size, beta) <= 13 / 12 * work * _us(torch, mode, *less, beta)


def test_tail_costs_less_than_a_slab(torch_cuda):  # noqa: F811
    """The last k mod 32 columns of a ragged product: eight of them cost less
    than the 32 that make k a multiple."""
    _us(torch_cuda, "fp64", 1777, 1650, 64, 0.0)
    assert _us(torch_cuda, "fp64", 1777, 1650, 40, 0.0) < _us(torch_cuda, "fp64", 1777, 1650, 64, 0.0)


@pytest.mark.parametrize("mode", ["fp64", "fp32"])
@pytest.mark.parametrize("m,n", [(37, 45), (150, 70), (1030, 777)])
def test_every_tail_length(torch_cuda, mode, m, n):  # noqa: F811
    """k = 1 .. 33 and one slab more, against FP64 on the host: an element is a
    sum of k products of numbers below 6 in chains of roundings, so its error is
    at most 36 k (k + 4) u."""
    torch = torch_cuda
    import paper_1801_04723_amd as S
    dt, u = (torch.float64, 2.0 ** -53) if mode == "fp64" else (torch.float32, 2.0 ** -24)
    g = torch.Generator().manual_seed(m)
    a, b = torch.randn(65, m + 1, generator=g, dtype=dt).clamp(-6, 6), torch.randn(n, 67, generator=g, dtype=dt).clamp(-6, 6)
    da, db = a.cuda(), b.cuda()
    for k in (*range(1, 34), 35, 63, 65):
        d = torch.empty(n, m, dtype=dt, device="cuda")
        S.gemm_cm(m, n, k, 1.0, da, m + 1, db, 67, 0.0, None, m, d, m, dtype=mode)
        want = b[:, :k].double() @ a[:k, :m].double()
        assert float((d.cpu().double() - want).abs().max()) <= 36 * k * (k + 4) * u, k
