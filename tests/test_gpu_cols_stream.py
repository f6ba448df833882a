"""Column subsets of matrices with many rows, where workgroups stay and take a row after the other: against the columns of
the dense matrix, over the edges of that form (words and waves of the bitmap, rounds of queries, rows that do not fit
the staging area, rows whose next entry is not their end, ends of the arrays)."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

POISON = 0x77


def _dense(rows, cols, keep, wide, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randint(1, 256, (rows, cols), device="cuda", generator=g, dtype=torch.int16)
    keep = keep if torch.is_tensor(keep) else torch.full((rows, 1), keep, device="cuda")
    w *= torch.rand((rows, cols), device="cuda", generator=g) < keep
    return w if wide else w.to(torch.uint8)


def _compressed(w, shift=0):
    """Bitmap, values (`shift` elements into a buffer of other bits), row offsets, all on the device."""
    b, v, r = orc.compress(w.cpu().numpy().view(np.uint16 if w.dtype == torch.int16 else np.uint8))
    bitmap = torch.zeros(endor.bitmap_bytes(*w.shape), dtype=torch.uint8, device="cuda")
    bitmap[:b.size] = torch.from_numpy(b).cuda()
    buf = torch.full((shift + v.size + 16,), POISON, dtype=w.dtype, device="cuda")
    buf[shift:shift + v.size] = torch.from_numpy(v.view(np.int16) if w.dtype == torch.int16 else v).cuda()
    return endor.DeviceMatrix(w.shape[0], w.shape[1], bitmap, buf[shift:shift + v.size], int(v.size)), torch.from_numpy(r).cuda()


def _check(w, sel, shift=0, out_shift=0, m=None, ro=None, want=None):
    if m is None:
        m, ro = _compressed(w, shift)
    rows, nsel = w.shape[0], sel.numel()
    buf = torch.full((out_shift + rows * nsel + 64,), POISON, dtype=w.dtype, device="cuda")
    out = buf[out_shift:out_shift + rows * nsel].view(rows, nsel)
    endor.decompress_cols(m, ro, sel, out=out)
    torch.cuda.synchronize()
    want = w[:, sel] if want is None else want
    assert torch.equal(out, want)
    assert torch.all(buf[:out_shift] == POISON) and torch.all(buf[out_shift + rows * nsel:] == POISON)


# rows, cols, keep, wide, columns asked: groups of 4 and 8 waves; words of the bitmap per row around a wave's and a
# workgroup's; rounds of 4, 6, 8, 12 queries, full and not; rows of a workgroup odd and even; values to the last unit.
# Each takes this form, and together all of its instantiations: test_cols_plan.py.
CASES = [(5500, 4096, 0.5, True, 1600), (5501, 4097, 0.7, True, 1537), (6143, 4159, 0.5, False, 1600), (6145, 16384, 0.44, True, 1409),
         (5600, 16320, 0.46, True, 3072), (5500, 16385, 0.5, True, 2048), (5700, 20011, 0.7, True, 5000), (5500, 32768, 0.46, True, 2049),
         (5777, 32705, 0.9, False, 6144), (9001, 3333, 0.95, False, 1536), (5503, 12345, 0.02, False, 3071),
         (5500, 8000, 0.0, False, 3000), (6500, 16400, 0.49, True, 2049), (5500, 20500, 0.6, True, 1281),
         (5501, 8000, 0.45, True, 3071), (5500, 20011, 0.7, True, 4000), (5500, 32705, 0.9, False, 2048), (5501, 32705, 0.9, False, 3000),
         (5500, 32705, 0.9, False, 4000)]
# of the tests below: rows, cols, keep, columns asked
ANY_ORDER, NOT_STAGED = (5600, 8000, 0.6, 2900), (5555, 16001, 2500)
OWN_ENTRY, IN_A_GRAPH = (5504, 6000, 0.5, 1600), (5520, 9000, 0.7, 2000)


@pytest.mark.parametrize("rows, cols, keep, wide, nsel", CASES, ids=str)
def test_rows_one_after_the_other(rows, cols, keep, wide, nsel):
    print(f"stream {rows}x{cols} keep {keep} wide {wide} nsel {nsel}", flush=True)
    w = _dense(rows, cols, keep, wide, rows + cols)
    sel = torch.randperm(cols, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))[:nsel].sort().values
    _check(w, sel, shift=(rows % 7), out_shift=rows % 5)


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
def test_any_order_repeats_and_indices_outside(wide):
    rows, cols, keep, nsel = ANY_ORDER
    w = _dense(rows, cols, keep, wide, 3)
    g = torch.Generator(device="cuda").manual_seed(2)
    sel = torch.randint(0, cols, (nsel,), device="cuda", generator=g)
    outside = torch.tensor([-1, cols, cols + 31, 1 << 40, -(1 << 50)], device="cuda")
    at = torch.tensor([0, 63, 64, 1499, nsel - 1], device="cuda")
    want = w[:, sel].clone()
    want[:, at] = POISON  # those columns of the output are left as they are
    sel[at] = outside
    _check(w, sel, want=want)


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
def test_rows_that_are_not_staged(wide):
    """Full rows among sparse ones (more values than the staging area holds), empty rows, and the last row."""
    rows, cols, nsel = NOT_STAGED
    keep = torch.full((rows, 1), 0.4 if wide else 0.8, device="cuda")
    keep[::97] = 1.0
    keep[5::101] = 0.0
    keep[-1] = 1.0
    _check(_dense(rows, cols, keep, wide, 4), torch.arange(7, 7 + nsel * 7, 7, device="cuda") % cols, shift=1)


def test_only_a_rows_own_entry_says_where_its_values_are():
    """Entries that are not in order: the next one is too small, too large, or another row's."""
    rows, cols, keep, nsel = OWN_ENTRY
    w = _dense(rows, cols, keep, True, 5)
    m, ro = _compressed(w)
    sel = torch.arange(0, nsel * 3, 3, device="cuda")
    order = torch.randperm(rows, device="cuda", generator=torch.Generator(device="cuda").manual_seed(6))
    # row i of another matrix has row order[i]'s bits and values: its offsets point anywhere
    bits = torch.zeros((rows, cols), dtype=torch.uint8, device="cuda")
    bits.copy_(w[order] != 0)
    flat = torch.zeros(endor.bitmap_bytes(rows, cols) * 8, dtype=torch.uint8, device="cuda")
    flat[:rows * cols] = bits.view(-1)
    weights = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device="cuda")
    bitmap = (flat.view(-1, 8) * weights).sum(dim=1, dtype=torch.int32).to(torch.uint8)
    m2 = endor.DeviceMatrix(rows, cols, bitmap, m.values, m.nnz)
    ro2 = torch.cat([ro[:-1][order], ro[-1:]])
    _check(w[order], sel, m=m2, ro=ro2)


def test_columns_in_a_hip_graph():
    rows, cols, most, nsel = IN_A_GRAPH
    ws = [_dense(rows, cols, k, True, 7 + i) for i, k in enumerate((0.5, 0.3, most))]
    ms = [_compressed(w) for w in ws]
    cap = max(m.nnz for m, _ in ms)
    bitmap, values, ro = torch.zeros_like(ms[0][0].bitmap), torch.zeros(cap, dtype=torch.int16, device="cuda"), torch.zeros_like(ms[0][1])
    sel, out = torch.arange(0, nsel * 4, 4, device="cuda"), torch.empty((rows, nsel), dtype=torch.int16, device="cuda")
    m = endor.DeviceMatrix(rows, cols, bitmap, values, cap)
    endor.decompress_cols(m, ro, sel, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        endor.decompress_cols(m, ro, sel, out=out)
    for w, (c, r) in list(zip(ws, ms)) + [(ws[0], ms[0])]:
        bitmap.copy_(c.bitmap)
        values[:c.nnz].copy_(c.values)
        ro.copy_(r)
        out.fill_(POISON)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, w[:, sel])
