"""The vector products where a segment's windows reach over an end of `values`: arrays of a few values, last
segments with none to nine, every 2-byte address; NaN patterns lie around the array.  Small integers, so the
sums are exact in fp32 whatever the order."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (rows, cols, values in all but the last segment, values in the last): segments of 2, 4, 6 and 8 steps
CASES = [(1, 600, 0, n) for n in (0, 1, 7, 8, 9, 10)] + [(2, 2000, 700, n) for n in (0, 1, 7, 8, 9)]
CASES += [(3, 4097, 3000, 1), (3100, 3073, 40000, 3)] + [(13000, 8200, 300000, 1)]


def _cuda16(x):
    return torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16)


@pytest.mark.parametrize("voff", [0, 1, 3])
@pytest.mark.parametrize("case", CASES, ids=str)
def test_ends_of_the_values(case, voff):
    rows, cols, many, last = case
    print(f"gemv ends {case} voff={voff}", flush=True)
    g = np.random.default_rng(rows + cols + last)
    n = rows * cols
    flat = np.zeros(n, np.float16)
    tail = min(60, n)
    if many:
        flat[g.choice(n - tail, min(many, (n - tail) // 2), replace=False)] = 3
        flat[:20] = 2                                       # a first byte with all its bits set
    if last:
        flat[n - tail + np.arange(last) * (tail // last)] = np.arange(1, last + 1)
    w = flat.reshape(rows, cols)
    x = g.integers(-4, 5, (2, cols)).astype(np.float16)
    c = endor.compress(w)
    buf = torch.full((c.nnz + 16,), 0x7E00, dtype=torch.int16, device="cuda")
    buf[voff:voff + c.nnz] = torch.from_numpy(c.values.view(np.int16)).cuda()
    m = endor.DeviceMatrix(rows, cols, torch.from_numpy(c.bitmap).cuda(), buf[voff:voff + c.nnz], c.nnz)
    y = endor.gemv_f16(m, torch.from_numpy(c.row_offsets).cuda(), _cuda16(x[0]))
    ws, _ = endor.build_offsets(m)
    Y = endor.gemm_f16(m, ws, _cuda16(x))
    torch.cuda.synchronize()
    ref = orc.gemm_f16(rows, cols, c.bitmap, c.values, x)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), ref[0])
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
