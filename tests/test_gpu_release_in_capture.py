"""Handles may be released at any time, also while a stream is being captured:
the capture goes on.  More handles than share one piece of pinned memory."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("count", [3, 300])
def test_release_while_capturing(count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1610_07902_amd as spv
    n = 1000
    at = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    ones = torch.ones(n, device="cuda")
    out = torch.zeros(16, device="cuda")

    def multiply(M):
        yi, yv, nnz = M.spmspv(at[:n:7].contiguous(), ones[:n:7].contiguous(), sorted_output=True)
        assert nnz == (n + 6) // 7 and bool((yv == 1.0).all())

    for k in range(2):   # the second time with what the first released
        handles = [spv.Matrix(n, n, at, at[:n].contiguous(), ones) for _ in range(count)]
        for M in handles[::50]:
            multiply(M)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out.add_(1.0)
            for M in handles[1:]:
                M.close()
            out.add_(1.0)
        for _ in range(2):
            graph.replay()
        multiply(handles[0])
        assert bool((out == 4.0 * (k + 1)).all())
        handles[0].close()
