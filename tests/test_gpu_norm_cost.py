"""The time of a small norm right behind the kernel that wrote the matrix, as the
refinement has it: a few round trips to memory."""
import ctypes

import pytest

from test_gpu_leafspec import torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def _graph_us(torch, fn, reps=20):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(reps):
            fn()
    for _ in range(3):
        g.replay()
    best = float("inf")
    for _ in range(8):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(5):
            g.replay()
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1) * 1e3 / (5 * reps))
    return best


@pytest.mark.parametrize("n", [192, 320, 384])
def test_small_norm_behind_its_writer(torch_cuda, n):  # noqa: F811
    """At most 6.7 us, what three launches (partial sums, sum, check) took; a
    launch in a graph takes about 2."""
    torch = torch_cuda
    import paper_1801_04723_amd as S
    frob = S.lib()["_ZN4spin5frob2EPKdlllPdS2_P12ihipStream_t"]
    frob.argtypes = [ctypes.c_void_p] + [ctypes.c_int64] * 3 + [ctypes.c_void_p] * 3
    a = torch.randn(n, n, dtype=torch.float64, device="cuda")
    b = a.clone()
    ws = torch.zeros(4096, dtype=torch.float64, device="cuda").data_ptr()

    def write():
        torch.mul(b, 1.0, out=a)

    def both():
        write()
        frob(a.data_ptr(), n, n, n, ws + 4096, ws + 256, torch.cuda.current_stream().cuda_stream)

    assert _graph_us(torch, both) - _graph_us(torch, write) <= 6.7


@pytest.mark.parametrize("m,n", [(1, 1), (3, 2), (64, 3), (65, 17), (1, 513), (5000, 1), (100, 33), (257, 129),
                                 (1000, 47), (33, 4100), (2050, 1030)])
def test_column_groups(torch_cuda, m, n):  # noqa: F811
    """Views whose columns fall into whole and partial groups, against FP64 sums:
    at most m n + 400 roundings of positive terms."""
    torch = torch_cuda
    import paper_1801_04723_amd as S
    frob = S.lib()["_ZN4spin5frob2EPKdlllPdS2_P12ihipStream_t"]
    frob.argtypes = [ctypes.c_void_p] + [ctypes.c_int64] * 3 + [ctypes.c_void_p] * 3
    g = torch.Generator(device="cuda").manual_seed(m + n)
    a = torch.randn(n, m + 3, dtype=torch.float64, device="cuda", generator=g)
    ws = torch.zeros(4096, dtype=torch.float64, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    got = set()
    for _ in range(3):
        assert frob(a.data_ptr(), m + 3, m, n, ws.data_ptr() + 4096, ws.data_ptr() + 256, s) == 0
        got.add(float(ws[32]))
    assert len(got) == 1
    want = float((a[:, :m].cpu() ** 2).sum())
    assert abs(got.pop() - want) <= (m * n + 400) * 2.0 ** -53 * want
