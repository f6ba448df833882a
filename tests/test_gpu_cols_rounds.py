"""Column subset: the number of queries around every edge of a thread's round, and outputs on both sides of the
sizes where their stores are streamed; rows gathered and staged, 16- and 8-bit values.  Bit for bit."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MB = 1 << 20
# (rows, cols, columns asked, keep): 3, 4 and 6 queries a thread; odd numbers; one row; then the outputs of 8 and 96 MB
CASES = [(3, 5000, n, 0.5) for n in (1, 255, 257, 767, 768, 769, 1023, 1024, 1025, 1535, 1536, 1537, 2048, 2049, 3073)]
CASES += [(1, 70001, 1537, 0.3), (700, 9001, 1538, 0.5), (2049, 4100, 4 * MB // 2049, 0.1), (2049, 4100, 4 * MB // 2049 + 1, 0.1),
          (7200, 7100, 48 * MB // 7200, 0.5), (7200, 7100, 48 * MB // 7200 + 1, 0.5)]
# short rows, of which few enough values are asked to gather them and enough to stage them; many of those, where workgroups stay
CASES += [(12000, 2500, 1100, 0.8), (5400, 2000, 1700, 0.95), (12000, 2500, 1500, 0.8), (12001, 2501, 1701, 0.7)]


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
@pytest.mark.parametrize("rows,cols,nsel,keep", CASES)
def test_cols_rounds(rows, cols, nsel, keep, wide):
    print(f"cols rounds rows={rows} cols={cols} nsel={nsel} keep={keep} wide={wide}", flush=True)
    g = np.random.default_rng(nsel)
    w = g.integers(1, 255, (rows, cols), dtype=np.uint8)
    w[g.random((rows, cols), dtype=np.float32) >= keep] = 0
    w = w.astype(np.uint16) if wide else w
    w[:, cols // 3: cols // 3 + 300] = 9                 # whole pieces of ones, several banks' worth
    w[rows // 2] = 7                                     # a row with more values than the others
    sel = np.sort(g.permutation(cols)[:nsel])
    if nsel > 2:
        sel[:2] = sel[1::-1]                             # out of order
        sel[-1] = sel[0]                                 # asked twice
    idx = sel.astype(np.int64)
    c = endor.compress(w)
    got = endor.decompress_cols(endor.to_device(c), torch.from_numpy(c.row_offsets).cuda(), torch.from_numpy(idx).cuda())
    assert np.array_equal(got.cpu().numpy().view(w.dtype).reshape(rows, nsel), w[:, sel])
