"""The exchange of partial sums in block-rows that are spread over the XCDs (the last T % 8): a reducer there may start before
its producers and hands the sum over to whoever arrives last.  libspqt_handover.so is the library with reducers that hand
over at once, so that path runs in every spread block-row.  The order of the sum is the same, so the results are those of
the product library bit for bit, and both leave the whole workspace, counters included, zero."""
import os

import numpy as np
import pytest

import oracle
from workloads import make_weights, make_x, quantile_threshold

pytestmark = pytest.mark.gpu

HEIGHT = {"g": 256, "cb": 256, "cbk": 256, "cb8": 128, "cb2": 512}


@pytest.fixture(scope="module")
def libs():
    import torch
    import paper_2511_04477_amd as spqt
    from paper_2511_04477_amd import binding
    product = spqt.lib()
    path = os.path.join(os.path.dirname(spqt.__file__), "libspqt_handover.so")
    assert os.path.exists(path), "libspqt_handover.so is not built (python -m paper_2511_04477_amd.build)"
    keep = binding.LIB_PATH
    binding.LIB_PATH, binding._lib = path, None
    try:
        other = binding.lib()
    finally:
        binding.LIB_PATH, binding._lib = keep, product

    def both(call):
        """call() with the product library, then with the other one."""
        out = []
        for L in (product, other):
            binding._lib = L
            try:
                out.append(call())
            finally:
                binding._lib = product
        return out
    return torch, spqt, both


def run(torch, spqt, layout, packed, M, K, x, idx, cnt, thr, mode, **shape):
    rows = x.shape[0] if x.dim() == 2 else 1
    y = torch.full((rows, M) if rows > 1 else (M,), float("nan"), dtype=torch.float32, device="cuda")
    ws = spqt.new_workspace(M, K, rows)
    if mode == "fused":
        if layout == "g" and rows > 1:
            shape.pop("waves", None)
            spqt.spqt_gemv_fused_rows(packed, M, K, x, thr, y, ws, **shape)
        else:
            getattr(spqt, "spqt_gemv_fused" if layout == "g" else f"spqt_{layout}_gemv_fused")(packed, M, K, x, thr, y, ws, **shape)
    else:
        name = "spqt_gemv" if layout == "g" else f"spqt_{layout}_gemv" + ("_rows" if rows > 1 and layout in ("cb8", "cb2") else "")
        lists = (idx, cnt) if mode == "list" else (None, None)
        getattr(spqt, name)(packed, M, K, x, *lists, y, ws, **shape)
    torch.cuda.synchronize()
    assert int(torch.count_nonzero(ws).item()) == 0, "the workspace must be all zeros between calls"
    return y.cpu().numpy()


@pytest.mark.parametrize("layout,rows,mode", [("g", 1, "list"), ("g", 1, "fused"), ("g", 1, "dense"), ("g", 2, "list"), ("g", 2, "fused"),
                                              ("g", 3, "list"), ("g", 4, "fused"), ("g", 4, "dense"), ("cb", 1, "list"), ("cb", 4, "dense"),
                                              ("cbk", 1, "fused"), ("cb8", 1, "list"), ("cb8", 4, "list"), ("cb2", 1, "fused"),
                                              ("cb2", 3, "dense")])
@pytest.mark.parametrize("T", [4, 9, 23])
def test_handed_over_sums(libs, layout, rows, mode, T):
    """T block-rows: all spread, one of nine, seven of 23 - workgroups per block-row around the 4 and 16 words that are collected
    at once, one wavefront per workgroup (several rounds of units per thread) and four."""
    torch, spqt, both = libs
    M, K = HEIGHT[layout] * T, 2560
    r = np.random.default_rng(7000 + T)
    if layout == "g":
        w = make_weights(M, K, 7001 + T)
        packed_np = spqt.spqt_pack(w["q_rowmajor"], w["scales"])
    else:
        W = np.tile(r.standard_normal((64, K)).astype(np.float32), (M // 64, 1)) * np.linspace(0.5, 1.5, M, dtype=np.float32)[:, None]
        packed_np = getattr(spqt, f"spqt_{layout}_quantize")(W)
    x_np = make_x(K, "laplace", 7002, batch=rows)
    thr = quantile_threshold(x_np, 0.5)
    packed = torch.from_numpy(packed_np).cuda()
    x = torch.from_numpy(x_np if rows > 1 else x_np[0].copy()).cuda()
    idx, cnt = torch.empty(K, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    spqt.spqt_gather(x, thr, idx, cnt)
    most = 16 if layout == "cb2" else 64
    shapes = [dict(), dict(splits=2), dict(splits=5), dict(splits=6), dict(splits=min(17, most)), dict(splits=min(18, most)), dict(splits=min(40, most))]
    if not (layout == "g" and mode == "fused" and rows > 1):
        shapes += [dict(splits=3, waves=1), dict(splits=min(20, most), waves=1)]
    for shape in shapes:
        print(f"hand-over {layout} rows={rows} {mode} T={T} {shape}", flush=True)
        a, b = both(lambda: run(torch, spqt, layout, packed, M, K, x, idx, cnt, thr, mode, **shape))
        assert np.array_equal(a, b), f"{shape}: {np.abs(a - b).max()}"
        if layout == "g":
            ref = oracle.gemv(w["q_rowmajor"], w["scales"], x_np, 0.0 if mode == "dense" else thr)
            assert np.all(np.abs(a.reshape(rows, M) - ref) <= 1e-2 + 2e-3 * np.abs(ref)), shape
