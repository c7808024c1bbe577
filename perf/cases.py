"""What is timed when the speed of this library is judged: the work a decoder running on it does.

A case is either a chain of GEMVs - `layers` decoder layers, each a few projections with weights of
their own - or the offline conversion of one matrix on the host.  A chain runs one of the ways the
library offers: "list" (spqt_gather, then the GEMV over the index list, per projection), "fused"
(threshold, compaction and GEMV in one launch) or "dense" (no list).  Serving loops replay the chain
as one HIP graph ("graph"); short scripts and tests call the binding directly ("eager").  Sizes are
those of the benchmark's configurations (7B, 8B, 13B and 70B projection shapes) and odd ones.

Weights are drawn on the GPU directly in the packed layouts that spqt.h and spqt_colblock.h state (any
byte is a valid pair of codes), enough of them per pass that they do not stay in the 256 MB cache;
activations are Laplace, Gaussian or SiLU(g)*u, thresholds calibrated on a separate draw as a model's
would be, so the kept count varies a little from layer to layer.
"""
import math

import numpy as np
import torch

import paper_2511_04477_amd as spqt

LAYOUTS = {
    # rows of a block-row, columns of a chunk, scale bytes at its head, bits of a code
    "g128": (256, 128, 512, 4),
    "g64": (256, 64, 512, 4),
    "cb": (256, 128, 2048, 4),
    "cbk": (256, 128, 2048, 4),
    "cb8": (128, 128, 1024, 8),
    "cb2": (512, 128, 4096, 2),
}


def _chain(name, layout, mode, projections, layers, sparsity, dist="laplace", rows=1, own=False, out="float32",
           graph=True):
    case = {"kind": "chain", "layout": layout, "mode": mode, "projections": projections, "layers": layers,
            "sparsity": sparsity, "dist": dist, "rows": rows, "own": own, "out": out, "graph": graph}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest configuration, called as a script or a test calls it: two launches, all latency
        _chain("small_eager", "g128", "list", "512x1024", 1, 0.5, "normal", graph=False),
        # direct calls on a matrix of no round size with groups of 64, several matrices in turn
        _chain("ragged_g64_eager", "g64", "list", "11001x4224", 4, 0.4, graph=False),
        # one token through Llama-3-8B's projections, a threshold and an index list per projection
        _chain("decoder_8b", "g128", "list",
               "4096x4096 1024x4096 1024x4096 4096x4096 14336x4096 14336x4096 4096x14336", 8, 0.5),
        # one token through Llama-2-7B's MLP with the one-launch entry point
        _chain("mlp_7b_one_launch", "g128", "fused", "11008x4096 11008x4096 4096x11008", 16, 0.4),
        # the benchmark's largest shapes, batch 1: the bandwidth-bound end
        _chain("mlp_70b", "g128", "list", "28672x8192 28672x8192 8192x28672", 3, 0.5),
        # the same with four activation rows on the union of their kept columns
        _chain("mlp_70b_rows4", "g128", "list", "28672x8192 8192x28672", 3, 0.7, rows=4),
        # a beam of two, every row its own kept set, one launch per projection, fp16 results
        _chain("beam2_8b_own_sets", "g128", "fused", "14336x4096 4096x14336", 12, 0.65, "silu_product", rows=2, own=True,
               out="float16"),
        # no sparsity at all: layers whose activations are not thresholded (13B shapes)
        _chain("dense_13b", "g128", "dense", "5120x5120 13824x5120 5120x13824", 6, 0.0),
        # the column-block layout, index list
        _chain("colblock_8b", "cb", "list", "4096x4096 14336x4096 4096x14336", 8, 0.5),
        # its K-quant flavour in one launch
        _chain("kquant_13b_one_launch", "cbk", "fused", "13824x5120 5120x13824", 6, 0.4),
        # its 8-bit flavour, index list, fp16 results
        _chain("w8_7b", "cb8", "list", "4096x4096 11008x4096 4096x11008", 4, 0.5, out="float16"),
        # the offline side: one matrix into the zigzag layout and back, on the host
        {"name": "pack_unpack", "kind": "pack", "group": 128, "M": 4096, "K": 4096},
    ]


def draw(rng):
    """A case of the same ranges: any layout, mode, number of rows and output type the entry points take."""
    if rng.random() < 0.08:
        M = int(round(2 ** rng.uniform(9, 12)))
        return {"kind": "pack", "group": rng.choice([128, 64]), "M": M, "K": 128 * rng.randint(8, 32)}
    layout = rng.choice(["g128"] * 6 + ["g64", "cb", "cb", "cbk", "cb8", "cb2"])
    mode = rng.choice(["list", "list", "fused", "dense"])
    rows = rng.choice([1, 1, 1, 2, 3, 4]) if layout in ("g128", "g64") else 1
    if layout in ("cb", "cbk", "cb8") and mode != "fused":
        rows = rng.choice([1, 1, 1, 2, 4])
    K = 128 * int(round(2 ** rng.uniform(3, math.log2(224))))
    M = int(round(2 ** rng.uniform(9, min(math.log2(28672), math.log2(235e6 / K)))))
    high = LAYOUTS[layout][0]
    if layout in ("cbk", "cb2") or rng.random() < 0.5:
        M = max(high, M // high * high)
    per_layer = M * K * LAYOUTS[layout][3] // 8
    graph = rng.random() < 0.8
    layers = max(1, min(24 if graph else 4, (360 << 20) // per_layer))
    sparsity = 0.0 if mode == "dense" else round(rng.uniform(0.2, 0.75), 2)
    return _chain(None, layout, mode, "%dx%d" % (M, K), layers, sparsity, rng.choice(["laplace", "normal", "silu_product"]),
                  rows, rows > 1 and layout in ("g128", "g64") and mode != "dense" and rng.random() < 0.5,
                  rng.choice(["float32", "float32", "float16"]), graph)


def _shapes(case):
    return [tuple(int(v) for v in p.split("x")) for p in case["projections"].split()]


# ------------------------------------------------------------------------------- inputs

def _values(dist, shape, gen):
    def normal():
        return torch.randn(shape, device="cuda", generator=gen)
    if dist == "normal":
        return normal()
    if dist == "silu_product":
        return torch.nn.functional.silu(normal()) * normal()
    u = torch.rand(shape, device="cuda", generator=gen) - 0.5
    return -torch.sign(u) * torch.log1p(-2 * u.abs().clamp(max=0.499999))


def _threshold(dist, sparsity, gen):
    if sparsity <= 0:
        return 0.0
    v = _values(dist, (1 << 16,), gen).half().float().abs().sort().values
    return float(v[int(sparsity * v.numel())])


def _packed(layout, M, K, gen):
    """Random codes and scales in the packed form of an M x K matrix; rows past M as the packers store them."""
    high, cols, head, bits = LAYOUTS[layout]
    T, n = -(-M // high), K // cols
    buf = torch.randint(0, 256, (T, n, head + cols * 128), dtype=torch.uint8, device="cuda", generator=gen)
    scales = (torch.rand((T, n, head // 2), device="cuda", generator=gen) * 0.015 + 0.005).half()
    if bits != 4:
        scales *= 0.1 if bits == 8 else 4.0
    if layout == "cbk":   # d and dmin of a column, then its 6-bit fields (already random)
        half = buf[:, :, :head].view(T, n, cols, 16)
        half[..., :4] = (scales.view(T, n, cols, 8)[..., :2] / 32).contiguous().view(torch.uint8)
    else:
        buf[:, :, :head] = scales.view(torch.uint8)
    last = M - (T - 1) * high
    if last < high:
        codes = buf[-1, :, head:].view(n, cols, 128)
        if bits == 4:
            if last % 2:
                codes[..., last // 2] = (codes[..., last // 2] & 15) | 0x80
            codes[..., (last + 1) // 2:] = 0x88
        else:
            codes[..., last:] = 128
        sc = buf[-1, :, :head].view(torch.float16)
        if layout in ("g128", "g64"):
            sc[:, last:] = 0
        else:
            sc.view(n, cols, -1)[..., -(-last // 32):] = 0
    return buf.reshape(-1)


def prepare(case, seed):
    if case["kind"] == "pack":
        r = np.random.default_rng(seed)
        q = r.integers(0, 256, (case["M"], case["K"] // 2), dtype=np.uint8)
        s = r.uniform(0.005, 0.02, (case["M"], case["K"] // case["group"])).astype(np.float16)
        return {"case": case, "q": q, "scales": s}
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rows, layers, K_of = case["rows"], case["layers"], {}
    out = getattr(torch, case["out"])
    steps, results, spaces = [], [], {}
    for M, K in _shapes(case):
        lead = (layers, rows) if rows > 1 else (layers,)
        x = _values(case["dist"], lead + (K,), gen).half()
        thr = _threshold(case["dist"], case["sparsity"], gen)
        y = torch.zeros(lead + (M,), dtype=out, device="cuda")
        idx = torch.zeros((layers, K), dtype=torch.int32, device="cuda")
        count = torch.zeros((layers, 1), dtype=torch.int32, device="cuda")
        masked = torch.zeros_like(x) if case["own"] and case["mode"] == "list" else None
        if (M, K) not in spaces:
            spaces[M, K] = spqt.new_workspace(M, K, rows)
        weights = [_packed(case["layout"], M, K, gen) for _ in range(layers)]
        steps.append((M, K, weights, x, thr, idx, count, masked, y, spaces[M, K]))
        results.append((y, idx, count) if case["mode"] == "list" else (y,))
    # layer by layer, each layer's projections in order
    order = [(s[0], s[1], s[2][i], s[3][i], s[4], s[5][i], s[6][i], None if s[7] is None else s[7][i], s[8][i], s[9])
             for i in range(layers) for s in steps]
    state = {"case": case, "order": order, "results": results, "graph": None}
    if case["graph"]:
        _pass(case, order[: len(steps)])          # kernels are loaded before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _pass(case, order)
        state["graph"] = graph
    return state


# --------------------------------------------------------------------------------- a pass

def _pass(case, order):
    layout, mode, rows, own = case["layout"], case["mode"], case["rows"], case["own"]
    group = 64 if layout == "g64" else 128
    for M, K, w, x, thr, idx, count, masked, y, ws in order:
        if mode == "fused":
            if rows > 1:
                spqt.spqt_gemv_fused_rows(w, M, K, x, thr, y, ws, own_sets=own, group=group)
            elif layout in ("g128", "g64"):
                spqt.spqt_gemv_fused(w, M, K, x, thr, y, ws, group=group)
            else:
                getattr(spqt, "spqt_%s_gemv_fused" % layout)(w, M, K, x, thr, y, ws)
            continue
        if mode == "list":
            if masked is not None:
                spqt.spqt_gather_rows(x, thr, idx, count, masked)
                x = masked
            else:
                spqt.spqt_gather(x, thr, idx, count)
        else:
            idx = count = None
        if layout in ("g128", "g64"):
            spqt.spqt_gemv(w, M, K, x, idx, count, y, ws, group=group)
        elif layout == "cb8" and rows > 1:
            spqt.spqt_cb8_gemv_rows(w, M, K, x, idx, count, y, ws)
        else:
            getattr(spqt, "spqt_%s_gemv" % layout)(w, M, K, x, idx, count, y, ws)


def run(state):
    case = state["case"]
    if case["kind"] == "pack":
        packed = spqt.spqt_pack(state["q"], state["scales"], case["group"])
        q, scales = spqt.spqt_unpack(packed, case["M"], case["K"], case["group"])
        return {"packed": packed, "q": q, "scales": scales.view(np.uint16)}
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _pass(case, state["order"])
    return state["results"]


# ----------------------------------------------------------------------- work, tolerance

def work(case):
    if case["kind"] == "pack":
        both = case["M"] * case["K"] // 2 + 2 * case["M"] * case["K"] // case["group"]
        return {"bytes": 4 * both, "flops": 0}
    high, cols, head, bits = LAYOUTS[case["layout"]]
    rows = case["rows"]
    total = flops = 0.0
    for M, K in _shapes(case):
        kept = K * (1 - case["sparsity"] ** rows)
        b = kept * M * bits / 8 + 2 * rows * K + rows * M * (2 if case["out"] == "float16" else 4)
        b += 2.0 * M * K / cols if case["layout"] in ("g128", "g64") else kept * M / 16
        if case["mode"] == "list":
            b += 4 * kept
            if case["own"]:
                b += 2 * rows * K
        total += b * case["layers"]
        flops += 2.0 * M * kept * rows * case["layers"]
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    # four times what the kernels differ by from the same product in 64 bits: 5e-6 (largest element
    # 1.3e-5) with 32-bit sums, 2e-4 (5e-4) where the result is rounded to fp16
    if case["out"] == "float16":
        return {"rel": 8e-4, "max": 2e-3}
    return {"rel": 2e-5, "max": 6e-5}
