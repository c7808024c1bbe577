"""The exchange of partial sums at the numbers of workgroups per block-row where its loads change (4, 8, 12 or 16 words at once, then
rounds of 16), in whole and in spread block-rows.  x holds small integers and scales are powers of two, so every sum is exact in
32 bits whatever its order: the outputs equal those of one workgroup per block-row bit for bit, and the workspace is left all zeros."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SPLITS = (2, 5, 6, 9, 10, 13, 14, 17, 18, 33, 34)


@pytest.mark.parametrize("T", [1, 8, 9])
@pytest.mark.parametrize("layout,rows,waves", [("g128", 1, 4), ("g128", 1, 1), ("g128", 2, 4), ("g128", 3, 8), ("g128", 4, 4), ("cb", 1, 4),
                                               ("cb", 3, 4), ("cb8", 1, 4), ("cb8", 3, 2), ("cb2", 1, 4)])
def test_any_number_of_workgroups_gives_the_same_sums(layout, rows, waves, T):
    import torch
    import paper_2511_04477_amd as spqt
    high, cols, head = {"g128": (256, 128, 512), "cb": (256, 128, 2048), "cb8": (128, 128, 1024), "cb2": (512, 128, 4096)}[layout]
    M, K = high * T - 3 * (layout == "g128"), 2304
    r = np.random.default_rng(100 * T + rows)
    chunks = r.integers(0, 256, (T, K // cols, head + cols * 128), dtype=np.uint8)
    chunks[:, :, :head] = np.exp2(r.integers(-3, 2, (T, K // cols, head // 2))).astype(np.float16).view(np.uint8)
    packed = torch.from_numpy(chunks.reshape(-1)).cuda()
    x = torch.from_numpy(r.integers(-4, 5, (rows, K)).astype(np.float16)).cuda()
    x = x[0].contiguous() if rows == 1 else x
    ws = spqt.new_workspace(M, K, rows)
    gemv = {"g128": spqt.spqt_gemv, "cb": spqt.spqt_cb_gemv, "cb8": spqt.spqt_cb8_gemv if rows == 1 else spqt.spqt_cb8_gemv_rows,
            "cb2": spqt.spqt_cb2_gemv}[layout]

    def run(splits):
        print(f"exchange {layout} rows={rows} waves={waves} T={T} splits={splits}", flush=True)
        y = torch.full((rows, M) if rows > 1 else (M,), float("nan"), dtype=torch.float32, device="cuda")
        gemv(packed, M, K, x, None, None, y, ws, splits=splits, waves=waves)
        torch.cuda.synchronize()
        assert int(torch.count_nonzero(ws).item()) == 0
        return y

    alone = run(1)
    assert bool(torch.isfinite(alone).all())
    for splits in SPLITS if layout != "cb2" else SPLITS[:7]:      # 2-bit: at most 16
        assert torch.equal(run(splits), alone), splits
