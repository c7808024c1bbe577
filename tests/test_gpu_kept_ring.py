"""One launch over the column-block layouts (kept_ring.hpp): kept columns come from a ring that a refill of 192 columns fills, and
the passes take 64 entries of it from slices that begin at any column - against the dequantized weights in 64-bit arithmetic,
|y_gpu - y_ref| <= 1e-2 + 2e-3 * |y_ref|."""
import numpy as np
import pytest

from workloads import make_fp_weights, make_x

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["cb", "cbk", "cb8", "cb2"])
@pytest.mark.parametrize("K,splits", [(128, 1), (640, 3), (2944, 1)])
def test_kept_columns_of_any_slice(layout, K, splits):
    import torch
    import paper_2511_04477_amd as spqt
    M = 512
    packed_np = getattr(spqt, f"spqt_{layout}_quantize")(make_fp_weights(M, K, 6300 + K))
    deq = getattr(spqt, f"spqt_{layout}_dequantize")(packed_np, M, K).astype(np.float64)
    packed, ws = torch.from_numpy(packed_np).cuda(), spqt.new_workspace(M, K)
    base = make_x(K, "normal", 6301)[0]
    base = np.where(np.abs(base) < 0.25, np.float16(0.25), base).astype(np.float16)
    # nothing; entries around half a pass, a pass and the ring's turn; runs behind stretches that keep nothing for several refills
    for n in sorted({min(n, K) for n in (0, 1, 31, 33, 64, 65, 127, 129, 500, 600, K)}):
        spread = np.unique(np.linspace(0, K - 1, n).astype(int)) if n else np.zeros(0, int)
        for name, cols in (("spread", spread), ("run", np.arange(n)), ("tail", np.arange(K - n, K))):
            x_np = np.zeros_like(base)
            x_np[cols] = base[cols]
            x = torch.from_numpy(x_np).cuda()
            y = torch.full((M,), float("nan"), device="cuda")
            print(f"{layout} K={K} splits={splits} n={n} {name}", flush=True)
            getattr(spqt, f"spqt_{layout}_gemv_fused")(packed, M, K, x, 0.125, y, ws, splits=splits)
            torch.cuda.synchronize()
            ref = deq @ x_np.astype(np.float64)
            err = np.abs(y.cpu().numpy().astype(np.float64) - ref)
            assert np.all(err <= 1e-2 + 2e-3 * np.abs(ref)), f"n={n} {name}: max err {np.nanmax(err):.3e}"


@pytest.mark.parametrize("layout", ["cb", "cbk", "cb8", "cb2"])
def test_dropped_columns_stay_out_of_empty_passes(layout):
    """Column 0 is dropped and its scales are infinite: a pass without entries points at it and must not multiply it."""
    import torch
    import paper_2511_04477_amd as spqt
    M, K = 512, 1024
    packed_np = getattr(spqt, f"spqt_{layout}_quantize")(make_fp_weights(M, K, 6400))
    deq = getattr(spqt, f"spqt_{layout}_dequantize")(packed_np, M, K).astype(np.float64)
    per_column = {"cb": 16, "cbk": 4, "cb8": 8, "cb2": 32}[layout]      # cbk: d and dmin, then the 6-bit fields
    chunk = {"cb": 18432, "cbk": 18432, "cb8": 17408, "cb2": 20480}[layout]
    for t in range(packed_np.size // (K // 128 * chunk)):
        at = t * (K // 128) * chunk
        packed_np[at:at + per_column] = np.full(per_column // 2, np.inf, dtype=np.float16).view(np.uint8)
    packed, ws = torch.from_numpy(packed_np).cuda(), spqt.new_workspace(M, K)
    x_np = np.zeros(K, dtype=np.float16)
    x_np[700:] = 0.5
    y = torch.full((M,), float("nan"), device="cuda")
    getattr(spqt, f"spqt_{layout}_gemv_fused")(packed, M, K, torch.from_numpy(x_np).cuda(), 0.125, y, ws, splits=1)
    torch.cuda.synchronize()
    deq[:, 0] = 0.0
    ref = deq @ x_np.astype(np.float64)
    err = np.abs(y.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= 1e-2 + 2e-3 * np.abs(ref)), float(np.nanmax(err))
