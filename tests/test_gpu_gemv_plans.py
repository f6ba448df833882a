"""The vector products in the forms their plans take at their edges: x in one panel that is just full and in
several, with the starts from the offset table and from the row offsets.  Small integers, so the sums are
exact; compared with the product in double precision on the same device."""
import pytest

import paper_2406_11674_amd as endor

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (rows, cols, right-hand sides): two that fill LDS to 200 bytes; one vector in two, three and more panels
CASES = [(4400, 24570, 2), (300, 24576, 2), (33, 16384, 3), (70, 12288, 4), (260, 49152, 1), (2000, 60001, 1), (300, 160000, 1)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_plans_at_their_edges_are_exact(case):
    rows, cols, nb = case
    print(f"gemv plans {case}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(rows + nb)
    w = torch.randint(1, 5, (rows, cols), device="cuda", generator=gen, dtype=torch.int16).half()
    w *= torch.rand((rows, cols), device="cuda", generator=gen) < 0.4
    x = torch.randint(-4, 5, (nb, cols), device="cuda", generator=gen).half()
    m, ws, ro = endor.compress_device(w.view(torch.int16), row_offsets=True)
    ref = x.double() @ w.double().t()
    assert torch.equal(endor.gemm_f16(m, ws, x).double(), ref)
    assert torch.equal(endor.gemv_f16(m, ro, x[0]).double(), ref[0])
