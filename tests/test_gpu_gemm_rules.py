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
])
def test_time_grows_with_the_work(torch_cuda, mode, size, less, beta):  # noqa: F811
    torch = torch_cuda
    _us(torch, mode, *less, beta)
    work = (size[0] * size[1] * size[2]) / (less[0] * less[1] * less[2])
    assert _us(torch, mode, *size, beta) <= 13 / 12 * work * _us(torch, mode, *less, beta)
