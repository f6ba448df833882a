"""The products for one to four right-hand sides: every segment length, rows whole and in parts, x in one
panel and in several, against the oracle.  Small integers throughout, so every partial sum is an integer
below 2^24, exact in fp32 whatever the order, and the results must be equal."""
import numpy as np
import pytest

import paper_2406_11674_amd as endor
from oracle import endor_oracle as orc

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _problem(rows, cols, nb, keep, voff):
    print(f"few rhs rows={rows} cols={cols} nb={nb} keep={keep} voff={voff}", flush=True)
    g = np.random.default_rng(rows * 31 + cols + nb)
    p = np.full(rows, keep, np.float32)
    p[3::17] = 1.0          # full rows: every byte's last value comes from the next window
    p[1:2] = 0.0            # an empty one
    w = np.zeros((rows, cols), np.float16)
    at = g.random((rows, cols), dtype=np.float32) < p[:, None]
    w[at] = g.integers(1, 5, int(at.sum()))
    x = g.integers(-4, 5, (nb, cols)).astype(np.float16)
    c = endor.compress(w)
    buf = torch.full((c.nnz + 16,), 0x7E00, dtype=torch.int16, device="cuda")          # NaN patterns around
    buf[voff:voff + c.nnz] = torch.from_numpy(c.values.view(np.int16)).cuda()
    m = endor.DeviceMatrix(rows, cols, torch.from_numpy(c.bitmap).cuda(), buf[voff:voff + c.nnz], c.nnz)
    return c, m, x


def _cuda16(x):
    return torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16)


GEMV = [(1, 1), (2, 7), (1, 8), (5, 9), (300, 511), (40, 513), (300, 1025), (17, 2049), (9, 4097),   # 2 and 4 steps a segment
        (260, 2561), (7, 3071), (3100, 3073),                                                       # 6 steps; rows whole
        (2, 40000), (3, 130001), (1, 1 << 20),                                                      # parts; x in panels
        (9000, 40), (130000, 12), (270000, 3)]                                                      # many items, many workgroups


@pytest.mark.parametrize("shape", GEMV, ids=str)
def test_gemv_forms_are_exact(shape):
    rows, cols = shape
    c, m, x = _problem(rows, cols, 1, 0.45, rows % 4)
    y = endor.gemv_f16(m, torch.from_numpy(c.row_offsets).cuda(), _cuda16(x[0]))
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(np.float64), orc.gemv_f16(rows, cols, c.bitmap, c.values, x[0]))


GEMM = [(1, 8, 1), (5, 9, 4), (70, 511, 3), (300, 1030, 2), (33, 4099, 4), (600, 5005, 3), (3200, 3001, 2),
        (2, 24500, 2), (3, 16384, 3), (1, 49152, 1),                  # x that just fits LDS
        (9000, 60, 1), (4096, 40, 2), (9000, 500, 1),                 # narrow, up to the most rows that are taken
        (9000, 60, 4), (2, 24577, 2), (5, 7, 3), (32770, 3100, 5)]    # left to the matrix cores


@pytest.mark.parametrize("shape", GEMM, ids=str)
def test_gemm_with_few_right_hand_sides_is_exact(shape):
    rows, cols, nb = shape
    c, m, x = _problem(rows, cols, nb, 0.45, rows % 4)
    ws, _ = endor.build_offsets(m)
    xs = torch.zeros((nb, cols + 3), dtype=torch.float16, device="cuda")  # rows of x apart, at any 2-byte address
    xs[:, 1:1 + cols] = _cuda16(x)
    Y = endor.gemm_f16(m, ws, xs[:, 1:1 + cols])
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.gemm_f16(rows, cols, c.bitmap, c.values, x))


@pytest.mark.parametrize("nb", [1, 2])
def test_longest_segments_are_exact(nb):
    """Segments of 4096 columns are for matrices of a hundred of them per compute unit: compared with
    the product in double precision on the same device (gemv and gemm with one, gemm with two)."""
    rows, cols = 13000, 8200
    print(f"longest segments nb={nb}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(nb)
    w = torch.randint(1, 5, (rows, cols), device="cuda", generator=gen).half()
    w *= torch.rand((rows, cols), device="cuda", generator=gen) < 0.45
    x = torch.randint(-4, 5, (nb, cols), device="cuda", generator=gen).half()
    m, ws, ro = endor.compress_device(w.view(torch.int16), row_offsets=True)
    ref = x.double() @ w.double().t()
    assert torch.equal(endor.gemm_f16(m, ws, x).double(), ref)
    if nb == 1:
        assert torch.equal(endor.gemv_f16(m, ro, x[0]).double(), ref[0])
