"""run() without a stream launches on torch's current stream, whichever that is."""
import pytest
import torch

from paper_1903_06498_amd import binding as B
from paper_1903_06498_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_run_takes_the_current_stream():
    side = torch.cuda.Stream()
    assert B.current_stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B.current_stream() == side.cuda_stream != torch.cuda.default_stream().cuda_stream
    assert B.current_stream() == torch.cuda.current_stream().cuda_stream
    # captured with the stream: the launches are in the graph, and a replay writes the output
    sb = B.StripeBlock(W.matmul_block(16, 24, 32, "f32", "f32"))
    a, b = W.seeded_tensor((16, 32), "f32", 0).cuda(), W.seeded_tensor((32, 24), "f32", 1).cuda()
    out, graph = torch.zeros((16, 24), device="cuda"), torch.cuda.CUDAGraph()
    sb.run([a, b], out)
    with torch.cuda.graph(graph):
        sb.run([a, b], out)
    want = a.double() @ b.double()
    tol = 32 * 2.0 ** -24 * (a.double().abs() @ b.double().abs())      # 32 fp32 additions
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert ((out.double() - want).abs() <= tol).all()
    sb.close()
