"""The calls whose speed this library is kept to, as a user's program makes them.

Everything goes through the public entry points of `paper_2406_11674_amd`, on inputs that are
resident on the GPU (the host-to-device pipeline apart, whose inputs are pinned host memory by
their nature).  The sizes are the library's own: the linear layers of OPT-66B and Llama2-70B at
the paper's 50 % sparsity, the keep sweep around it, and odd sizes of the parity tests' kind.

A program that decompresses or multiplies keeps its compressed weights, its output buffers, its
workspace and its tables from call to call, so `prepare` makes those; activations, selections and
dense matrices to be compressed come with every call, so they differ from state to state.
"""
import math

import torch

import paper_2406_11674_amd as endor

SIGMA = 0.02  # standard deviation of the weights that are kept

# one Llama2-70B decoder layer: q, k, v, o, gate, up, down
LLAMA2_70B_LAYER = ((8192, 8192), (1024, 8192), (1024, 8192), (8192, 8192), (28672, 8192), (28672, 8192), (8192, 28672))


def listed():
    return [
        # The smallest call in use: one 1024 x 1024 projection, where latency and launches count.
        {"name": "decompress_1024sq", "op": "decompress", "rows": 1024, "cols": 1024, "keep": 0.5, "bytes": 2},
        # The headline: all linear weights of a decoder layer ahead of its forward pass, one batched call.
        {"name": "decompress_llama2_70b_layer", "op": "layer", "rows": 0, "cols": 0, "keep": 0.5, "bytes": 2},
        # A heavily pruned down projection: nearly all of the traffic is the dense output.
        {"name": "decompress_down_keep10", "op": "decompress", "rows": 8192, "cols": 28672, "keep": 0.1, "bytes": 2},
        # The 8-bit variant (pruning joined with quantization) on the OPT-66B feed-forward matrix.
        {"name": "decompress_u8_fc2", "op": "decompress", "rows": 9216, "cols": 36864, "keep": 0.5, "bytes": 1},
        # A weight decompressed again for every generated token, its offset table kept; odd ragged
        # size, so that rows straddle bitmap words and the last tile is partial.
        {"name": "redecompress_odd", "op": "redecompress", "rows": 5003, "cols": 3171, "keep": 0.7, "bytes": 2},
        # Activation sparsity, up side: a tenth of the gate projection's rows.
        {"name": "rows_gate_tenth", "op": "rows", "rows": 28672, "cols": 8192, "keep": 0.5, "bytes": 2, "share": 0.1},
        # Activation sparsity, down side: a tenth of the down projection's columns.
        {"name": "cols_down_tenth", "op": "cols", "rows": 8192, "cols": 28672, "keep": 0.5, "bytes": 2, "share": 0.1},
        # The other direction: a pruned matrix that is already on the GPU is brought into the format.
        {"name": "compress_gate", "op": "compress", "rows": 28672, "cols": 8192, "keep": 0.5, "bytes": 2},
        # Decode: one token against the compressed down projection.
        {"name": "gemv_down", "op": "gemv", "rows": 8192, "cols": 28672, "keep": 0.5, "bytes": 2},
        # A full small batch (16 tokens: batched decode, speculative verification, a short prefill).
        {"name": "gemm16_gate", "op": "gemm", "rows": 28672, "cols": 8192, "keep": 0.5, "bytes": 2, "nb": 16},
        # A few tokens against an ordinary odd-sized matrix, sparser than half.
        {"name": "gemm3_odd", "op": "gemm", "rows": 4099, "cols": 5005, "keep": 0.3, "bytes": 2, "nb": 3},
        # Offloaded inference: the compressed OPT-66B feed-forward matrix lives in pinned host memory
        # and is decompressed while its row blocks arrive.
        {"name": "pipeline_fc1", "op": "pipeline", "rows": 36864, "cols": 9216, "keep": 0.5, "bytes": 2, "blocks": 4},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any operation, sizes from a small projection to the largest listed matrix,
    aligned (multiples of 64, as model shapes are) or odd, any density in use."""
    op = rng.choice(["decompress", "decompress", "redecompress", "rows", "cols", "compress", "gemv", "gemv", "gemm", "gemm",
                     "pipeline"])
    while True:
        rows, cols = _log_uniform(rng, 512, 36864), _log_uniform(rng, 512, 36864)
        if rng.random() < 0.6:
            rows, cols = max(64, rows // 64 * 64), max(64, cols // 64 * 64)
        if rows * cols <= 36864 * 9216:
            break
    case = {"op": op, "rows": rows, "cols": cols, "keep": round(rng.uniform(0.1, 0.9), 2), "bytes": 2}
    if op in ("decompress", "redecompress", "rows", "cols", "compress") and rng.random() < 0.3:
        case["bytes"] = 1
    if op in ("rows", "cols"):
        case["share"] = round(rng.uniform(0.05, 0.5), 2)
    if op == "gemm":
        case["nb"] = rng.randint(1, 16)
    if op == "pipeline":
        case["blocks"] = rng.randint(1, 6)
    return case


# ---------------------------------------------------------------- inputs

def _shapes(case):
    return LLAMA2_70B_LAYER if case["op"] == "layer" else ((case["rows"], case["cols"]),)


def _generator(seed, index=0):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + index)


def _dense(case, shape, gen):
    """A pruned weight: normal values (fp16 bit patterns) or 8-bit codes, kept at random places, the
    others all-zero patterns.  No kept element is zero.  The matrix keeps exactly round(keep * n)
    elements, as a pruner with a given ratio leaves it."""
    rows, cols = shape
    keep = torch.rand((rows, cols), device="cuda", generator=gen) < case["keep"]
    surplus = int(keep.sum()) - round(case["keep"] * rows * cols)
    if surplus != 0:  # a few thousand at most: flipped at regular distances
        at = (keep if surplus > 0 else ~keep).view(-1).nonzero().view(-1)
        keep.view(-1)[at[::at.numel() // abs(surplus)][:abs(surplus)]] = surplus < 0
        del at
    if case["bytes"] == 2:
        w = (torch.randn((rows, cols), device="cuda", generator=gen) * SIGMA).half()
        w[w == 0] = SIGMA
        return w.masked_fill_(~keep, 0).view(torch.int16)
    w = torch.randint(1, 256, (rows, cols), device="cuda", generator=gen, dtype=torch.uint8)
    return w * keep


def _compressed(dense):
    """The bitmap format in plain torch: bit e & 7 of byte e >> 3, whole 64-bit words; packed values."""
    flat = dense.reshape(-1)
    mask = flat != 0
    padded = torch.zeros(endor.bitmap_bytes(*dense.shape) * 8, dtype=torch.uint8, device="cuda")
    padded[:flat.numel()] = mask
    bits = padded.view(-1, 8)
    bitmap = bits[:, 0].clone()
    for k in range(1, 8):
        bitmap |= bits[:, k] << k
    values = flat[mask]
    return endor.DeviceMatrix(dense.shape[0], dense.shape[1], bitmap, values, values.numel())


def _row_offsets(dense):
    offsets = torch.zeros(dense.shape[0] + 1, dtype=torch.int64, device="cuda")
    torch.cumsum((dense != 0).sum(dim=1), 0, out=offsets[1:])
    return offsets


def _selection(case, gen):
    """The active neurons of one token: a sorted random subset."""
    of = case["rows"] if case["op"] == "rows" else case["cols"]
    count = max(1, int(of * case["share"]))
    return torch.randperm(of, device="cuda", generator=gen)[:count].sort().values


def _activations(case, gen):
    nb = case.get("nb", 1)
    return torch.randn((nb, case["cols"]), device="cuda", generator=gen).half()


def _element(case):
    return torch.int16 if case["bytes"] == 2 else torch.uint8


def prepare(case, seed):
    op = case["op"]
    gen = _generator(seed)
    state = {"op": op}
    if op == "layer":
        state["mats"] = [_compressed(_dense(case, s, _generator(seed, i))) for i, s in enumerate(_shapes(case))]
        state["outs"] = [torch.empty(s, dtype=torch.int16, device="cuda") for s in _shapes(case)]
        state["workspace"] = torch.empty(endor.batch_workspace_bytes(state["mats"]), dtype=torch.uint8, device="cuda")
        return state
    rows, cols = case["rows"], case["cols"]
    dense = _dense(case, (rows, cols), gen)
    if op == "compress":
        state["dense"] = dense
        return state
    state["m"] = m = _compressed(dense)
    if op == "pipeline":
        host = endor.Compressed(rows, cols, m.bitmap.cpu().numpy(), m.values.cpu().numpy(), _row_offsets(dense).cpu().numpy())
        del state["m"], m, dense
        blobs = endor.row_blocks(host, case["blocks"])
        out = torch.empty((rows, cols), dtype=_element(case), device="cuda")
        state["blobs"] = blobs
        state["out"] = out
        state["views"] = [out[b.row_begin:b.row_begin + b.rows] for b in blobs]
        state["compute"] = torch.cuda.Stream()
        state["pipeline"] = endor.Pipeline.for_blobs(blobs, torch.cuda.Stream(), state["compute"],
                                                     copy_stream2=torch.cuda.Stream())
        return state
    if op in ("decompress", "redecompress"):
        state["out"] = torch.empty((rows, cols), dtype=_element(case), device="cuda")
        state["workspace"] = torch.empty(endor.workspace_bytes(rows, cols), dtype=torch.uint8, device="cuda")
        if op == "redecompress":
            endor.build_offsets(m, state["workspace"])
    if op in ("rows", "cols"):
        state["row_offsets"] = _row_offsets(dense)
        state["sel"] = sel = _selection(case, gen)
        shape = (sel.numel(), cols) if op == "rows" else (rows, sel.numel())
        state["out"] = torch.empty(shape, dtype=_element(case), device="cuda")
    if op == "gemv":
        state["row_offsets"] = _row_offsets(dense)
        state["x"] = _activations(case, gen)[0]
        state["y"] = torch.empty(rows, dtype=torch.float32, device="cuda")
    if op == "gemm":
        state["workspace"], _ = endor.build_offsets(m)
        state["x"] = _activations(case, gen)
        state["y"] = torch.empty((case["nb"], rows), dtype=torch.float32, device="cuda")
        state["scratch"] = torch.empty(endor.gemm_scratch_bytes(rows, cols, case["nb"]), dtype=torch.uint8, device="cuda")
    return state


# ---------------------------------------------------------------- one pass

def run(state):
    op = state["op"]
    if op == "layer":
        endor.decompress_batch(state["mats"], outs=state["outs"], workspace=state["workspace"])
        return state["outs"]
    if op == "decompress":
        return endor.decompress(state["m"], out=state["out"], workspace=state["workspace"])
    if op == "redecompress":
        return endor.decompress_with_offsets(state["m"], state["workspace"], out=state["out"])
    if op == "rows":
        return endor.decompress_rows(state["m"], state["row_offsets"], state["sel"], out=state["out"])
    if op == "cols":
        return endor.decompress_cols(state["m"], state["row_offsets"], state["sel"], out=state["out"])
    if op == "compress":
        m, _, row_offsets = endor.compress_device(state["dense"], row_offsets=True)
        return {"bitmap": m.bitmap, "values": m.values, "row_offsets": row_offsets}
    if op == "gemv":
        return endor.gemv_f16(state["m"], state["row_offsets"], state["x"], y=state["y"])
    if op == "gemm":
        return endor.gemm_f16(state["m"], state["workspace"], state["x"], Y=state["y"], scratch=state["scratch"])
    # the pipeline computes on a stream of its own; the program goes on with the result on its stream
    state["compute"].wait_stream(torch.cuda.current_stream())
    state["pipeline"].run(state["blobs"], state["views"])
    torch.cuda.current_stream().wait_stream(state["compute"])
    return state["out"]


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    op, keep, e = case["op"], case["keep"], case["bytes"]
    n = sum(r * c for r, c in _shapes(case))
    rows, cols = case["rows"], case["cols"]
    compressed = n / 8 + keep * n * e
    if op in ("decompress", "redecompress", "layer", "compress"):
        return {"bytes": compressed + n * e + (8 * (rows + 1) if op == "compress" else 0), "flops": 0}
    if op == "pipeline":  # crosses the host link, is read from device memory again, and expanded
        return {"bytes": compressed + n * e, "flops": 0}
    if op == "rows":
        part = max(1, int(rows * case["share"])) / rows
        return {"bytes": part * (compressed + n * e + 16 * rows), "flops": 0}
    if op == "cols":
        # every bit of the bitmap (a rank needs the bits before it) and the selected values alone
        part = max(1, int(cols * case["share"])) / cols
        return {"bytes": n / 8 + part * (keep * n * e + n * e + 8 * cols) + 8 * rows, "flops": 0}
    nb = case.get("nb", 1)
    return {"bytes": compressed + nb * (2 * cols + 4 * rows), "flops": 2.0 * nb * keep * n}


def tolerance(case):
    """Moved patterns are the same bit for bit.  The products are sums of exact fp16 products in
    fp32, whose order is free."""
    return {"rel": 2e-6, "max": 2e-5} if case["op"] in ("gemv", "gemm") else "exact"


def exact(case, seed):
    """The products in 64 bits from the dense matrix; moved patterns have no rounding to compare."""
    if case["op"] not in ("gemv", "gemm"):
        return None
    gen = _generator(seed)
    w = _dense(case, (case["rows"], case["cols"]), gen).view(torch.float16).double()
    y = _activations(case, gen).double() @ w.t()
    return y[0] if case["op"] == "gemv" else y
