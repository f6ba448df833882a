"""Column subset whose output rows begin inside cache lines: rows gathered and staged, with and without room for
the queries that are counted from the line's start, and outputs at every kind of address.  Bit for bit, and nothing
outside the output is written."""
import pytest

import paper_2406_11674_amd as endor

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (rows, cols, columns asked, keep): outputs of 32 MB and more gathered, of 96 MB and more staged
# (test_cols_plan.py says which form each takes)
CASES = [(5500, 9000, n, 0.15) for n in (3071, 3072, 3073, 3136, 4545, 4609, 6143)]     # a row of 6-query rounds: full, one over
CASES += [(9300, 13001, n, 0.5) for n in (5569, 6081, 6144, 6145)]                      # staged, 4-query rounds
CASES += [(70000, 800, 767, 0.9), (1, 262144, 262143, 0.4)]                             # short rows; one row of 512 KB
CASES += [(30000, 3000, 1700, 0.8)]                                                     # short rows, staged


@pytest.mark.parametrize("case,off", [(c, off) for c in CASES for off in (0, 1, 37, 64) if off == 37 or c[0] * c[2] < 40_000_000], ids=str)
def test_rows_that_begin_inside_lines(case, off):
    rows, cols, nsel, keep = case
    print(f"cols lines {case} off={off}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(nsel)
    w = torch.randint(1, 30000, (rows, cols), device="cuda", generator=gen, dtype=torch.int16)
    w *= torch.rand((rows, cols), device="cuda", generator=gen) < keep
    sel = torch.randperm(cols, device="cuda", generator=gen)[:nsel].sort().values
    sel[:2] = sel[:2].flip(0)
    m, _, ro = endor.compress_device(w, row_offsets=True)
    buf = torch.full((rows * nsel + 256,), 77, dtype=torch.int16, device="cuda")
    out = buf[off:off + rows * nsel].view(rows, nsel)
    endor.decompress_cols(m, ro, sel, out=out)
    assert torch.equal(out, w[:, sel])
    assert bool((buf[:off] == 77).all()) and bool((buf[off + rows * nsel:] == 77).all())
    sel[5] = -1                                       # not a column: its place stays as it is
    sel[nsel - 1] = cols
    buf.fill_(55)
    endor.decompress_cols(m, ro, sel, out=out)
    ref = w[:, sel.clamp(0, cols - 1)]
    ref[:, 5] = 55
    ref[:, nsel - 1] = 55
    assert torch.equal(out, ref)
