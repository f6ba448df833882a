"""The binding's idea of the current stream is torch's, on the default stream and inside a stream context,
and a call without a stream argument runs there.  (Its streams are taken behind the pipeline's timing test.)"""
import pytest

import paper_2406_11674_amd as endor
from paper_2406_11674_amd import binding

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_current_stream_handle():
    assert binding._stream_handle(None) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream_handle(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
        w = torch.zeros((64, 64), dtype=torch.int16, device="cuda")
        w[::3, ::5] = 7
        m, _, _ = endor.compress_device(w)
        out = endor.decompress(m)
    assert binding._stream_handle(side) == side.cuda_stream
    assert binding._stream_handle(None) == torch.cuda.current_stream().cuda_stream != side.cuda_stream
    side.synchronize()
    assert torch.equal(out, w)
