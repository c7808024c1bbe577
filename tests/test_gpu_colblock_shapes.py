"""Default launch shapes and workgroup placement of the column-block kernels: block-rows that do not divide over the 8 XCDs,
numbers of workgroups per block-row that are no power of two, one and several workgroups per CU, slices around one
pass - against the dequantized weights in 64-bit arithmetic, |y_gpu - y_ref| <= 1e-2 + 2e-3 * |y_ref|."""
import numpy as np
import pytest

from workloads import make_fp_weights, make_x, quantile_threshold

pytestmark = pytest.mark.gpu

HEIGHT = {"cb": 256, "cbk": 256, "cb8": 128, "cb2": 512}


@pytest.mark.parametrize("layout", sorted(HEIGHT))
@pytest.mark.parametrize("T,K", [(1, 128), (9, 1024), (20, 2048), (33, 1152), (71, 512), (130, 384), (300, 128)])
def test_block_rows_over_xcds(layout, T, K):
    import torch
    import paper_2511_04477_amd as spqt
    M = HEIGHT[layout] * T - (19 if layout in ("cb", "cb8") else 0)
    W = np.tile(make_fp_weights(256, K, 6100 + T), (-(-M // 256), 1))[:M] * np.linspace(0.5, 1.5, M, dtype=np.float32)[:, None]
    packed_np = getattr(spqt, f"spqt_{layout}_quantize")(W)
    deq = getattr(spqt, f"spqt_{layout}_dequantize")(packed_np, M, K).astype(np.float64)
    x_np = make_x(K, "laplace", 6101 + T)
    thr = quantile_threshold(x_np, 0.5)
    xd = x_np[0].astype(np.float64)
    ref = {"dense": deq @ xd, "list": deq @ np.where(np.abs(xd) < thr, 0.0, xd)}
    ref["fused"] = ref["list"]
    packed, x = torch.from_numpy(packed_np).cuda(), torch.from_numpy(np.ascontiguousarray(x_np[0])).cuda()
    idx, cnt = torch.empty(K, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    spqt.spqt_gather(x, thr, idx, cnt)
    ws = spqt.new_workspace(M, K)
    gemv, fused = getattr(spqt, f"spqt_{layout}_gemv"), getattr(spqt, f"spqt_{layout}_gemv_fused")
    for splits in (0, 3, 5):
        for mode in ("list", "fused", "dense"):
            print(f"{layout} T={T} K={K} splits={splits} {mode}", flush=True)
            y = torch.full((M,), float("nan"), device="cuda")
            if mode == "fused":
                fused(packed, M, K, x, thr, y, ws, splits=splits)
            elif mode == "list":
                gemv(packed, M, K, x, idx, cnt, y, ws, splits=splits)
            else:
                gemv(packed, M, K, x, None, None, y, ws, splits=splits)
            torch.cuda.synchronize()
            err = np.abs(y.cpu().numpy().astype(np.float64) - ref[mode])
            assert np.all(err <= 1e-2 + 2e-3 * np.abs(ref[mode])), f"{layout} {mode} splits={splits}: max err {np.nanmax(err):.3e}"
