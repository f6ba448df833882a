"""The device compressor's one pass over the dense matrix, which large 16-byte aligned matrices take: against the
oracle's Algorithm 1, and against the two passes that the same matrix takes from an unaligned address.  Collected
late, as it takes streams of torch's pool."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc
from paper_2406_11674_amd import binding

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

POISON = 0x7FFF
MIN_FP16, MIN_U8 = 40 << 20, 160 << 20  # elements from which on it is taken


def _matrix(rows, cols, keep, wide, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randint(1, 65536 if wide else 256, (rows, cols), device="cuda", generator=g, dtype=torch.int32)
    if keep < 1:
        w *= torch.rand((rows, cols), device="cuda", generator=g) < keep
    return w.to(torch.int16) if wide else w.to(torch.uint8)


def _expect(dense):
    return orc.compress(dense.cpu().numpy().view(np.uint16 if dense.dtype == torch.int16 else np.uint8))


def _call(dense, values, capacity, want_rows=True, stream=None):
    """The C entry on buffers full of other bits: bitmap, values, row offsets, table, count; nothing is waited for."""
    rows, cols = dense.shape
    bitmap = torch.full((endor.bitmap_bytes(rows, cols),), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.full((endor.workspace_bytes(rows, cols),), 0xFF, dtype=torch.uint8, device="cuda")
    ro = torch.full((rows + 1,), -1, dtype=torch.int64, device="cuda") if want_rows else None
    nnz = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    fn = binding.lib().endor_compress_device if dense.dtype == torch.int16 else binding.lib().endor_compress_device_u8
    s = (stream or torch.cuda.current_stream())
    if stream is not None:
        stream.wait_stream(torch.cuda.current_stream())
    assert fn(rows, cols, dense.data_ptr(), bitmap.data_ptr(), values.data_ptr() if capacity else None, capacity, ws.data_ptr(),
              ws.numel(), ro.data_ptr() if want_rows else None, nnz.data_ptr(), s.cuda_stream) == 0
    return bitmap, ro, ws, nnz


def _table(ws, n):
    """The entries of the table, without the padding between its parts."""
    chunks = -(-n // (1 << 20))
    w = ws.view(torch.int32)
    at = ((4 * chunks + 255) & ~255) // 4
    return torch.cat([w[:chunks], w[at:at + 257 * chunks]])


# ragged (a last tile that ends inside a 16-byte unit, and blocks that end inside a round); whole tiles only; the smallest;
# rows of 4 (1024 start in every tile); rows longer than a chunk
SHAPES = [(5003, 8447, 0.5, True), (5003, 8447, 0.0, True), (5003, 8447, 1.0, True), (10241, 4096, 0.9, True),
          (MIN_FP16 // 4, 4, 0.3, True), (37, 1500001, 0.03, True), (12289, 13653, 0.5, False), (MIN_U8 // 640, 640, 1.0, False),
          (12289, 13653, 0.02, False)]


@pytest.mark.parametrize("rows, cols, keep, wide", SHAPES, ids=str)
def test_one_pass_matches_oracle_and_two_passes(rows, cols, keep, wide):
    print(f"one pass {rows}x{cols} keep {keep} wide {wide}", flush=True)
    n = rows * cols
    assert n >= (MIN_FP16 if wide else MIN_U8)
    dense = _matrix(rows, cols, keep, wide, rows + cols)
    b, v, r = _expect(dense)
    shifted = torch.empty(n + 1, dtype=dense.dtype, device="cuda")
    shifted[1:] = dense.view(-1)
    unaligned = shifted[1:].view(rows, cols)
    tables = []
    for d in (dense, unaligned):
        values = torch.full((v.size + 64,), POISON if wide else 0x7F, dtype=dense.dtype, device="cuda")
        bitmap, ro, ws, nnz = _call(d, values, v.size)
        torch.cuda.synchronize()
        assert int(nnz) == v.size and torch.all(values[v.size:] == (POISON if wide else 0x7F))
        assert np.array_equal(values[:v.size].cpu().numpy().view(v.dtype), v)
        bm = bitmap.cpu().numpy()
        assert np.array_equal(bm[:b.size], b) and not bm[b.size:].any()
        assert np.array_equal(ro.cpu().numpy(), r)
        tables.append(_table(ws, n))
    assert torch.equal(*tables)


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
def test_one_pass_keeps_to_the_capacity(wide):
    rows, cols = (5003, 8447) if wide else (12289, 13653)
    dense = _matrix(rows, cols, 0.4, wide, 5)
    _, v, _ = _expect(dense)
    poison = POISON if wide else 0x7F
    first = torch.from_numpy(v.view(np.int16) if wide else v).cuda()
    # values from every kind of address; room for all, one less, a part of a unit, none
    for shift, room in ((0, v.size), (1, v.size - 1), (3, v.size // 2), (7, 5), (5, 1), (2, 0)):
        print("capacity", shift, room, flush=True)
        buf = torch.full((shift + room + 64,), poison, dtype=dense.dtype, device="cuda")
        _, _, _, nnz = _call(dense, buf[shift:], room, want_rows=False)
        torch.cuda.synchronize()
        assert int(nnz) == v.size
        assert torch.all(buf[:shift] == poison) and torch.all(buf[shift + room:] == poison)
        assert torch.equal(buf[shift:shift + room], first[:room])


def test_one_pass_beside_other_work():
    """Calls on two streams at once, beside products on a third.  (How many workgroups run from the start is up to the dispatch;
    the next test holds compute units for that, and test_compress_plan.py replays every order on the host.)"""
    dense = [_matrix(5003, 8447, 0.5, True, 8), _matrix(12289, 13653, 0.5, False, 9)]
    want = [_expect(d) for d in dense]
    a = torch.randn((4096, 4096), device="cuda").half()
    side = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for _ in range(3):
        got = []
        values = [torch.empty(w[1].size, dtype=d.dtype, device="cuda") for d, w in zip(dense, want)]
        torch.cuda.synchronize()
        with torch.cuda.stream(side[2]):
            for _ in range(8):
                p = a @ a
        for d, val, s in zip(dense, values, side):
            got.append(_call(d, val, val.numel(), stream=s))
        torch.cuda.synchronize()
        for (bitmap, ro, _, nnz), val, (b, v, r) in zip(got, values, want):
            assert int(nnz) == v.size and np.array_equal(val.cpu().numpy().view(v.dtype), v)
            assert np.array_equal(bitmap.cpu().numpy()[:b.size], b) and np.array_equal(ro.cpu().numpy(), r)
        del p


@pytest.mark.parametrize("held_rows", [24, 250])
@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
def test_one_pass_begins_on_some_of_the_compute_units(wide, held_rows):
    """Vector products on another stream hold a compute unit for every row (all of its LDS), 0.2 ms at a time: longer than the
    compressor waits for its last workgroups.  It begins with the others, and these share what is left when they start:
    noted by a build for that, 232 workgroups to the end, and 6 that become 256 over seven spans.  (Several streams: some
    pairs of them share a hardware queue, and then nothing is held.)"""
    rows, cols = (9001, 8447) if wide else (16385, 13653)
    dense = _matrix(rows, cols, 0.5, wide, held_rows)
    b, v, r = _expect(dense)
    held = _matrix(held_rows, 2000000 if held_rows < 100 else 1000000, 0.5, True, 1)
    m, _, held_ro = endor.compress_device(held, row_offsets=True)
    x = torch.zeros(held.shape[1], device="cuda").half()
    y = torch.empty(held_rows, dtype=torch.float32, device="cuda")
    poison = POISON if wide else 0x7F
    side = [torch.cuda.Stream() for _ in range(4)]
    for k in (1, 2, 3):
        print("held rows", held_rows, "stream", k, flush=True)
        values = torch.full((v.size + 64,), poison, dtype=dense.dtype, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(side[0]):
            for _ in range(4):
                endor.gemv_f16(m, held_ro, x, y=y)
        bitmap, ro, ws, nnz = _call(dense, values, v.size, stream=side[k])
        torch.cuda.synchronize()
        assert int(nnz) == v.size and torch.all(values[v.size:] == poison)
        assert np.array_equal(values[:v.size].cpu().numpy().view(v.dtype), v)
        assert np.array_equal(bitmap.cpu().numpy()[:b.size], b) and np.array_equal(ro.cpu().numpy(), r)
        ws2, _ = endor.build_offsets(endor.DeviceMatrix(rows, cols, bitmap, values[:v.size], v.size))
        torch.cuda.synchronize()
        assert torch.equal(_table(ws, rows * cols), _table(ws2, rows * cols))


def test_one_pass_in_a_hip_graph_replays_correctly():
    rows, cols = 5003, 8447
    inputs = [_matrix(rows, cols, k, True, 20 + i) for i, k in enumerate((0.5, 0.2, 0.8))]
    want = [_expect(d) for d in inputs]
    dense = inputs[0].clone()
    values = torch.empty(max(w[1].size for w in want), dtype=torch.int16, device="cuda")
    bitmap = torch.empty(endor.bitmap_bytes(rows, cols), dtype=torch.uint8, device="cuda")
    ws = torch.empty(endor.workspace_bytes(rows, cols), dtype=torch.uint8, device="cuda")
    ro = torch.empty(rows + 1, dtype=torch.int64, device="cuda")
    nnz = torch.empty(1, dtype=torch.int64, device="cuda")

    def call(stream):
        assert binding.lib().endor_compress_device(rows, cols, dense.data_ptr(), bitmap.data_ptr(), values.data_ptr(), values.numel(),
                                                   ws.data_ptr(), ws.numel(), ro.data_ptr(), nnz.data_ptr(), stream.cuda_stream) == 0

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    call(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(torch.cuda.current_stream())
    for d, (b, v, r) in list(zip(inputs, want)) + [(inputs[0], want[0])]:
        dense.copy_(d)
        for t in (values, bitmap, ws, ro, nnz):
            t.fill_(0x5A)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(nnz) == v.size and np.array_equal(values[:v.size].cpu().numpy().view(np.uint16), v)
        assert np.array_equal(bitmap.cpu().numpy()[:b.size], b) and np.array_equal(ro.cpu().numpy(), r)
        ws2, _ = endor.build_offsets(endor.DeviceMatrix(rows, cols, bitmap, values, v.size))
        torch.cuda.synchronize()
        assert torch.equal(_table(ws, rows * cols), _table(ws2, rows * cols))
