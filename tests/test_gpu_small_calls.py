"""Decompression of small matrices in one kernel, a quarter of a tile per wave: around the edges of quarters,
tiles, workgroups and chunks, and on both sides of the size where two kernels take over; values and outputs
off their 16-byte boundaries.  Output and offset table are compared bit for bit."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [1, 63, 1023, 1024, 1025, 3072, 4095, 4097, 15 * 1024 + 1, 16 * 1024, (1 << 20) - 1, (1 << 20) + 1025, 3 * (1 << 20) - 4096,
         (1 << 22) - 1023, 1 << 22, (1 << 22) + 1]


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
@pytest.mark.parametrize("n", SIZES)
def test_small_decompress(n, wide):
    print(f"small decompress n={n} wide={wide}", flush=True)
    g = np.random.default_rng(n)
    dt = np.uint16 if wide else np.uint8
    tt = torch.int16 if wide else torch.uint8
    keep = (0.5, 0.08, 0.93)[n % 3]
    w = (g.integers(1, 255, (1, n)) * (g.random((1, n)) < keep)).astype(dt)
    w[0, n // 3: n // 3 + 2048] = 9                     # quarters with all bits set
    c = endor.compress(w)
    vbuf = torch.full((c.nnz + 16,), 77, dtype=tt, device="cuda")
    obuf = torch.full((n + 32,), 55, dtype=tt, device="cuda")
    ws = torch.empty(endor.workspace_bytes(1, n), dtype=torch.uint8, device="cuda")
    bitmap = torch.from_numpy(c.bitmap).cuda()
    table = torch.from_numpy(endor.build_offsets_host(c)).view(torch.uint8)
    for voff, ooff in ((0, 0), (3, 8), (1, 5)):
        vbuf.fill_(77)
        vbuf[voff:voff + c.nnz] = torch.from_numpy(c.values.view(np.int16 if wide else np.uint8)).cuda()
        obuf.fill_(55)
        ws.fill_(0xA5)
        m = endor.DeviceMatrix(1, n, bitmap, vbuf[voff:voff + c.nnz], c.nnz)
        endor.decompress(m, out=obuf[ooff:ooff + n], workspace=ws)
        torch.cuda.synchronize()
        got = obuf.cpu().numpy().view(dt)
        assert np.array_equal(got[ooff:ooff + n], w[0]), (voff, ooff)
        assert np.all(got[:ooff] == 55) and np.all(got[ooff + n:] == 55)
        nc = -(-n // (1 << 20))
        pad = -(-4 * nc // 256) * 256
        mine = ws.cpu()
        assert torch.equal(mine[:4 * nc], table[:4 * nc])
        assert torch.equal(mine[pad:pad + 4 * 257 * nc], table[pad:pad + 4 * 257 * nc])
    if wide and n < 1 << 20:
        assert np.array_equal(orc.decompress(1, n, c.bitmap, c.values).view(dt).reshape(1, n), w)
