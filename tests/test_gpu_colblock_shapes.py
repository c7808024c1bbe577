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


@pytest.mark.parametrize("layout,mode,rows,T,refused,K", [("cb", "list", 1, 129, 128, 4096), ("cb", "fused", 1, 257, 256, 1920),
                                                          ("cb", "dense", 1, 513, 384, 512), ("cb", "list", 4, 257, 256, 4096),
                                                          ("cbk", "list", 1, 257, 256, 512), ("cb8", "list", 1, 129, 128, 4096),
                                                          ("cb8", "fused", 1, 257, 256, 1920), ("cb8", "dense", 2, 257, 256, 512)])
def test_tall_matrices_run_without_a_workspace(layout, mode, rows, T, refused, K):
    """With T block-rows a call that brings no workspace, or one that is too small, runs with one workgroup per block-row; with `refused`
    it is an error.  The sums of two launch shapes differ by the rounding of fp32 sums: below 1e-5 of the result."""
    import torch
    import paper_2511_04477_amd as spqt
    high, head = HEIGHT[layout], 1024 if layout == "cb8" else 2048
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6200 + T)
    x = torch.randn((rows, K) if rows > 1 else (K,), device="cuda", generator=gen).half()
    idx, cnt = torch.empty(K, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    spqt.spqt_gather(x, 0.6, idx, cnt)

    def call(M, packed, ws):
        y = torch.full((rows, M) if rows > 1 else (M,), float("nan"), device="cuda")
        if mode == "fused":
            getattr(spqt, f"spqt_{layout}_gemv_fused")(packed, M, K, x, 0.6, y, ws)
        else:
            name = f"spqt_{layout}_gemv" + ("_rows" if layout == "cb8" and rows > 1 else "")
            getattr(spqt, name)(packed, M, K, x, *((idx, cnt) if mode == "list" else (None, None)), y, ws)
        torch.cuda.synchronize()
        return y.double()

    for t in (T, refused):
        M = high * t
        packed = torch.randint(0, 256, (t * (K // 128), head + 128 * 128), dtype=torch.uint8, device="cuda", generator=gen)
        scales = (torch.rand((packed.shape[0], head // 2), device="cuda", generator=gen) * 0.01 + 0.003).half()
        packed[:, :head] = scales.view(torch.uint8)
        packed = packed.reshape(-1)
        ref = call(M, packed, spqt.new_workspace(M, K, rows))
        for ws in (None, torch.zeros(256, dtype=torch.uint8, device="cuda")):
            print(f"without workspace {layout} {mode} rows={rows} T={t} K={K} {ws is None}", flush=True)
            if t == T:
                assert float((call(M, packed, ws) - ref).norm() / ref.norm()) < 1e-5
            else:
                with pytest.raises(spqt.SpqtError):
                    call(M, packed, ws)
