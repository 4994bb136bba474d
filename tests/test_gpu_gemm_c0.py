"""C0 in the epilogue of the 256 x 256 BF16 and bf16x3 tiles: read ahead of its
use, also where the result takes its place and at the tiles' edges, and at no
more than the cost of streaming it.
"""
import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["bf16", "bf16x3"])
@pytest.mark.parametrize("m,n,k,pad", [(3588, 3585, 516, 4), (4096, 4096, 512, 0), (3844, 4095, 1028, 0)])
def test_result_in_the_place_of_c0(torch_cuda, mode, m, n, k, pad):  # noqa: F811
    """Equal, bit for bit, to strips too narrow for the large tiles."""
    torch = torch_cuda
    import paper_1801_04723_amd as S
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    lda, ldb, ldd = m + pad, k + pad, m + pad + 1
    a = torch.randn(k, lda, device="cuda", generator=g)
    b = torch.randn(n, ldb, device="cuda", generator=g)
    c = torch.randn(n, ldd, device="cuda", generator=g)
    d, e = c.clone(), c.clone()
    S.gemm_cm(m, n, k, -1.0, a, lda, b, ldb, 0.5, d, ldd, d, ldd, dtype=mode)
    for j in range(0, n, 512):
        w = min(512, n - j)
        S.gemm_cm(m, w, k, -1.0, a, lda, b[j:], ldb, 0.5, c[j:], ldd, e[j:], ldd, dtype=mode)
    assert torch.equal(d, e)


@pytest.mark.parametrize("mode", ["bf16", "bf16x3"])
@pytest.mark.parametrize("m,n,k", [(3072, 3584, 512), (6144, 6144, 1024)])
def test_c0_costs_its_stream(torch_cuda, mode, m, n, k):  # noqa: F811
    """C0 is 4 m n bytes; at 1.5 TB/s, a third of what a copy reaches, its
    reading may take that long over the product without it."""
    torch = torch_cuda
    import paper_1801_04723_amd as S
    a, b, c = (torch.randn(x, y, device="cuda") for x, y in ((k, m), (n, k), (n, m)))
    d = torch.empty(n, m, device="cuda")

    def us(beta):
        best = float("inf")
        for _ in range(7):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(10):
                S.gemm_cm(m, n, k, -1.0, a, m, b, k, beta, c, m, d, m, dtype=mode)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1) * 100.0)
        return best

    us(1.0)
    assert us(1.0) <= us(0.0) + 4.0 * m * n / 1.5e6
