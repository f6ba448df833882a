"""The one-kernel decompression captured into a HIP graph.  Collected after the pipeline's timing test: how
well that one's copies overlap depends on which streams of torch's pool it gets, and this file takes one."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc
from paper_2406_11674_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

POISON = 0x7FFF


def test_small_decompress_in_a_hip_graph_replays_correctly():
    """The one-kernel form looks at the bitmap's kind of memory on the host; captured, it is one kernel
    node, which reads what the buffers hold when it is replayed."""
    rows, cols = 700, 1000
    cs = [endor.compress(synth.pruned_fp16(rows, cols, 0.5, seed=40 + i)) for i in range(3)]
    nnz = max(c.nnz for c in cs)
    bitmap = torch.zeros(endor.bitmap_bytes(rows, cols), dtype=torch.uint8, device="cuda")
    values = torch.zeros(nnz, dtype=torch.int16, device="cuda")
    m = endor.DeviceMatrix(rows, cols, bitmap, values, nnz)
    out = torch.empty((rows, cols), dtype=torch.int16, device="cuda")
    ws = torch.empty(endor.workspace_bytes(rows, cols), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    endor.decompress(m, out=out, workspace=ws, stream=side)                    # warm-up outside capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        endor.decompress(m, out=out, workspace=ws, stream=torch.cuda.current_stream())
    for c in cs + cs[:1]:
        bitmap.copy_(torch.from_numpy(c.bitmap))
        values[:c.nnz].copy_(torch.from_numpy(c.values.view(np.int16)))
        out.fill_(POISON)
        ws.fill_(0xFF)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint16), orc.decompress(rows, cols, c.bitmap, c.values))
