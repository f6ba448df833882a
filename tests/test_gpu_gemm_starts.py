"""Where the rows' values start in the product on the matrix cores: rows that begin at words, tiles and chunks of the
bitmap, groups of rows over many chunks, more than 256 chunks before a group, empty matrices.  Small integers: every sum is
exact in fp32, so the result is the reference's bit for bit."""
import pytest

import paper_2406_11674_amd as endor

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# rows, cols, keep: rows at every word; at every tile; at every chunk, in 15, 16 and 17 rows; several chunks to a row;
# up to 64 chunks between the first and the last row of a group, which one wave scans, and 65; 300 chunks
CASES = [(130, 64, 0.5), (70, 4096, 0.3), (35, 1 << 20, 0.1), (17, 1 << 20, 0.3), (33, (1 << 20) + 64, 0.02), (16, 4 << 20, 0.05),
         (19, (4 << 20) + (1 << 18), 0.05), (19, (4 << 20) + (5 << 16), 0.05), (18, (4 << 20) + 70001, 0.05), (79, 4 << 20, 0.01), (2000, 513, 0.0), (65, 65537, 1.0)]


@pytest.mark.parametrize("nb", [8, 16])
@pytest.mark.parametrize("rows, cols, keep", CASES, ids=str)
def test_rows_start_where_their_values_do(rows, cols, keep, nb):
    print(f"gemm starts {rows}x{cols} keep {keep} nb {nb}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    w = torch.randint(1, 4, (rows, cols), device="cuda", generator=g, dtype=torch.int16).to(torch.float16)
    w *= torch.rand((rows, cols), device="cuda", generator=g) < keep
    x = torch.randint(-1, 2, (nb, cols), device="cuda", generator=g, dtype=torch.int16).to(torch.float16)
    m, ws, _ = endor.compress_device(w.view(torch.int16))
    y = endor.gemm_f16(m, ws, x)
    want = torch.zeros((nb, rows), dtype=torch.float64, device="cuda")
    for a in range(0, cols, 1 << 20):
        want += x[:, a:a + (1 << 20)].double() @ w[:, a:a + (1 << 20)].double().t()
    torch.cuda.synchronize()
    assert torch.equal(y.double(), want)
