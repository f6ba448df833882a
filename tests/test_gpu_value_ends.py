"""Decompression where the array of values begins and ends inside 16-byte units, as all arrays but one in eight (fp16)
do at their end: the first and last tiles of every kernel that stages values, against the oracle."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

POISON = 0x77


def _case(rows, cols, keep, wide, drop):
    g = np.random.default_rng(rows * 31 + cols + drop)
    w = g.integers(1, 256, (rows, cols)).astype(np.uint16 if wide else np.uint8)
    if wide:
        w |= 0x3C00
    w[g.random((rows, cols)) >= keep] = 0
    flat = w.reshape(-1)
    flat[np.flatnonzero(flat)[:drop]] = 0  # the count, and with it the end of the array, moves element by element
    return w


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
@pytest.mark.parametrize("rows, cols, keep", [(1, 5, 1.0), (3, 4097, 0.9), (64, 64, 0.02), (70, 1024, 0.7), (1100, 4096, 0.15), (1100, 4095, 0.8)], ids=str)
def test_values_that_begin_and_end_inside_units(rows, cols, keep, wide):
    """A tile, two, the one-kernel form, and (1100 rows) the two kernels with little and with full staging."""
    unit = 8 if wide else 16
    for drop in range(0, unit, 1 if rows < 1000 else 3):
        shift = (3 * drop + (wide and 1)) % unit  # elements in front of the array: other alignments of its start
        w = _case(rows, cols, keep, wide, min(drop, rows * cols - 1))
        b, v, r = orc.compress(w)
        print(f"ends {rows}x{cols} wide {wide} drop {drop} shift {shift} nnz {v.size}", flush=True)
        dt = torch.int16 if wide else torch.uint8
        buf = torch.full((shift + v.size + 40,), POISON, dtype=dt, device="cuda")
        buf[shift:shift + v.size] = torch.from_numpy(v.view(np.int16) if wide else v).cuda()
        bitmap = torch.zeros(endor.bitmap_bytes(rows, cols), dtype=torch.uint8, device="cuda")
        bitmap[:b.size] = torch.from_numpy(b).cuda()
        m = endor.DeviceMatrix(rows, cols, bitmap, buf[shift:shift + v.size], int(v.size))
        ws, ro = endor.build_offsets(m, row_offsets=True)
        out = endor.decompress_with_offsets(m, ws)
        small = endor.decompress(m)
        sel = torch.tensor(sorted({0, rows // 2, rows - 1}), dtype=torch.int64, device="cuda")
        part = endor.decompress_rows(m, ro, sel)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(w.dtype), w)
        assert np.array_equal(small.cpu().numpy().view(w.dtype), w)
        assert np.array_equal(part.cpu().numpy().view(w.dtype), w[sel.cpu().numpy()])
