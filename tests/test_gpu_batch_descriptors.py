"""A batch finds the matrix and the tile of every wave: counts of matrices around the launch group's, sizes around a
word's, a tile's and a chunk's edges, each tile's last words."""
import pytest

import paper_2406_11674_amd as endor

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# elements: part of a word, a word and one, a tile less one, one, and one and one; a chunk, and a tile and a bit more; three chunks
SIZES = [5, 63, 64, 65, 4095, 4096, 4097, 4160, 1 << 20, (1 << 20) + 4096 + 1, 3 * (1 << 20) - 63, 12289, 70000, 1, 8191, 1048575]


@pytest.mark.parametrize("wide", [True, False], ids=["fp16", "u8"])
@pytest.mark.parametrize("count", [1, 2, 3, 15, 16, 17, 33])
def test_every_matrix_of_a_batch(count, wide):
    print(f"batch of {count} wide={wide}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(count)
    dense, mats = [], []
    for i in range(count):
        n = SIZES[(7 * i + count) % len(SIZES)]
        w = torch.randint(1, 256, (1, n), device="cuda", generator=g, dtype=torch.int16)
        w *= torch.rand((1, n), device="cuda", generator=g) < (0.5, 0.1, 0.9)[i % 3]
        w = w if wide else w.to(torch.uint8)
        dense.append(w)
        mats.append(endor.compress_device(w)[0])
    outs = [torch.full_like(w, 0x55) for w in dense]
    endor.decompress_batch(mats, outs=outs)
    ws = endor.build_offsets_batch(mats)
    again = endor.decompress_batch_with_offsets(mats, ws)
    torch.cuda.synchronize()
    for i, w in enumerate(dense):
        assert torch.equal(outs[i].view_as(w), w) and torch.equal(again[i].view(w.dtype).view_as(w), w), (i, w.numel())
