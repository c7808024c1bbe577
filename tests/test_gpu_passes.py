"""GPU parity of the passes shared by the group-layout kernels (pass.hpp) where they can go wrong: entries around the 64 slots
of a pass and the groups a pass takes, stretches that keep nothing longer than one refill of the one-launch kernel (256
columns), block-rows that do not divide evenly over the 8 XCDs, workgroups of 8 wavefronts for 3 and 4 rows - against the
oracle, |y_gpu - y_ref| <= 1e-2 + 2e-3 * |y_ref| - and the rounding of the matrix-core sums against 64-bit arithmetic."""
import numpy as np
import pytest

import oracle
from workloads import make_weights, make_x, quantile_threshold

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    import paper_2511_04477_amd as spqt
    assert torch.cuda.is_available(), "these tests need the MI355X"
    spqt.lib()
    return torch, spqt, torch.device("cuda:0")


def run(gpu, w, x_np, thr, mode, group=128, splits=0, own=False):
    torch, spqt, dev = gpu
    M, K = w["q_rowmajor"].shape[0], w["q_rowmajor"].shape[1] * 2
    packed = torch.from_numpy(spqt.spqt_pack(w["q_rowmajor"], w["scales"], group)).to(dev)
    x = torch.from_numpy(np.ascontiguousarray(x_np)).to(dev)
    rows = x.shape[0]
    y = torch.full((rows, M), float("nan"), dtype=torch.float32, device=dev)
    ws = spqt.new_workspace(M, K, rows)
    xx, yy = (x, y) if rows > 1 else (x[0], y[0])
    if mode == "fused":
        if rows > 1:
            spqt.spqt_gemv_fused_rows(packed, M, K, xx, thr, yy, ws, own_sets=own, group=group, splits=splits)
        else:
            spqt.spqt_gemv_fused(packed, M, K, xx, thr, yy, ws, group=group, splits=splits)
    else:
        idx = torch.empty(K, dtype=torch.int32, device=dev)
        cnt = torch.zeros(1, dtype=torch.int32, device=dev)
        if mode == "list":
            spqt.spqt_gather(xx, thr, idx, cnt)
        else:
            idx = cnt = None
        spqt.spqt_gemv(packed, M, K, xx, idx, cnt, yy, ws, group=group, splits=splits)
    torch.cuda.synchronize()
    return y.cpu().numpy()


def check(got, ref, what):
    err = np.abs(got.astype(np.float64) - ref)
    assert np.all(err <= 1e-2 + 2e-3 * np.abs(ref)), f"{what}: max err {np.nanmax(err):.3e}"


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
@pytest.mark.parametrize("group", [128, 64])
def test_pass_edges(gpu, rows, group):
    """One workgroup walks the whole matrix, so a wavefront sees every pass length: n kept columns spread over the columns
    (many groups per pass), in one run (one group per pass), and behind a stretch that keeps nothing."""
    M, K = 256, 2048
    w = make_weights(M, K, 5100 + rows, group=group)
    base = make_x(K, "normal", 5101, batch=rows)
    base = np.where(np.abs(base) < 0.25, np.float16(0.25), base).astype(np.float16)
    for n in (0, 1, 63, 64, 65, 129, 257, 600):
        spread = np.unique(np.linspace(0, K - 1, n).astype(int)) if n else np.zeros(0, int)
        for name, cols in (("spread", spread), ("run", np.arange(n)), ("tail", np.arange(K - n, K))):
            x = np.zeros_like(base)
            x[:, cols] = base[:, cols]
            ref = oracle.gemv(w["q_rowmajor"], w["scales"], x, 0.125, group=group)
            for mode in ("list", "fused"):
                print(f"pass edges rows={rows} group={group} n={n} {name} {mode}", flush=True)
                check(run(gpu, w, x, 0.125, mode, group, splits=1), ref, f"n={n} {name} {mode}")


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
@pytest.mark.parametrize("mode", ["dense", "list", "fused"])
def test_short_pass_behind_a_full_one_is_exact(gpu, rows, mode):
    """Slices of 96 columns: a pass of 64 entries, then one of 32, whose other slots must not keep the x of the first.  Small
    integers and scales that are powers of two: every product and sum is exact, so the outputs are the oracle's bit for bit."""
    M, K = 300, 384
    w = make_weights(M, K, 5300)
    w["scales"] = (2.0 ** np.random.default_rng(5301).integers(-3, 1, w["scales"].shape)).astype(np.float16)
    x = np.random.default_rng(5302 + rows).integers(1, 9, (rows, K)).astype(np.float16)
    ref = oracle.gemv(w["q_rowmajor"], w["scales"], x, 0.0)
    print(f"short pass rows={rows} {mode}", flush=True)
    assert np.array_equal(run(gpu, w, x, 0.0, mode, splits=1).astype(np.float64), ref)


@pytest.mark.parametrize("rows", [1, 2, 4])
def test_half_passes(gpu, rows):
    """Slices that end around 32 entries past a whole number of passes (the second half of such a pass has no products): four
    wavefronts with 31 to 33, 95 to 97 entries each; and dense slices of 32 and 96 columns."""
    M, K = 256, 640
    w = make_weights(M, K, 5150 + rows)
    base = make_x(K, "normal", 5151, batch=rows)
    base = np.where(np.abs(base) < 0.25, np.float16(0.25), base).astype(np.float16)
    for n in (4, 124, 127, 128, 129, 132, 380, 384, 385, 388):
        for name, cols in (("spread", np.unique(np.linspace(0, K - 1, n).astype(int))), ("run", np.arange(n))):
            x = np.zeros_like(base)
            x[:, cols] = base[:, cols]
            ref = oracle.gemv(w["q_rowmajor"], w["scales"], x, 0.125)
            for mode in ("list", "fused"):
                print(f"half passes rows={rows} n={n} {name} {mode}", flush=True)
                check(run(gpu, w, x, 0.125, mode, splits=1), ref, f"n={n} {name} {mode}")
    for Kd in (128, 384):
        wd = make_weights(M, Kd, 5160 + rows)
        xd = make_x(Kd, "normal", 5161, batch=rows)
        print(f"half passes rows={rows} dense K={Kd}", flush=True)
        check(run(gpu, wd, xd, 0.0, "dense", splits=1), oracle.gemv(wd["q_rowmajor"], wd["scales"], xd, 0.0), f"dense K={Kd}")


@pytest.mark.parametrize("rows", [1, 2, 3, 4])
def test_passes_end_at_any_sixteen(gpu, rows):
    """Slices of 15 to 17, 31 to 33 and 47 to 49 entries, and of as many behind a full pass (the products of the sixteens that a pass does not
    reach are left out): four wavefronts take a quarter of the list each.  Exact numbers, so the outputs are the oracle's bit for bit."""
    M, K = 256, 640
    w = make_weights(M, K, 5180)
    w["scales"] = (2.0 ** np.random.default_rng(5181).integers(-3, 1, w["scales"].shape)).astype(np.float16)
    base = np.random.default_rng(5182 + rows).integers(1, 9, (rows, K)).astype(np.float16)
    for each in (1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 80, 81, 112, 113):
        x = np.zeros_like(base)
        x[:, : 4 * each] = base[:, : 4 * each]
        ref = oracle.gemv(w["q_rowmajor"], w["scales"], x, 0.5)
        for mode in ("list", "fused"):
            print(f"sixteens rows={rows} each={each} {mode}", flush=True)
            assert np.array_equal(run(gpu, w, x, 0.5, mode, splits=1).astype(np.float64), ref), (each, mode)


@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("K,splits", [(128, 1), (384, 2), (640, 3), (1152, 5), (2944, 1)])
def test_one_launch_slices_of_any_column(gpu, rows, K, splits):
    """One launch: the slices are columns, not whole units of 64, so they begin and end anywhere inside a unit and a group."""
    w = make_weights(256, K, 5170 + K)
    x = make_x(K, "laplace", 5171 + K, batch=rows)
    for sparsity in (0.0, 0.5, 0.98):
        thr = quantile_threshold(x, sparsity) if sparsity else 0.0
        print(f"any column rows={rows} K={K} splits={splits} sparsity={sparsity}", flush=True)
        check(run(gpu, w, x, thr, "fused", splits=splits), oracle.gemv(w["q_rowmajor"], w["scales"], x, thr), f"K={K} sparsity={sparsity}")


@pytest.mark.parametrize("group", [128, 64])
@pytest.mark.parametrize("rows", [1, 2, 3, 4])
def test_dropped_groups_stay_out(gpu, rows, group):
    """All columns of the first groups are dropped and the scales of group 0 are infinite: slices and refills that keep nothing take
    passes without entries, which must not multiply those scales."""
    M, K = 512, 1024
    w = make_weights(M, K, 5180, group=group)
    x = np.zeros((rows, K), dtype=np.float16)
    x[:, 700:] = make_x(K, "normal", 5181, batch=rows)[:, 700:]
    ref = oracle.gemv(w["q_rowmajor"], w["scales"], x, 0.125, group=group)
    w["scales"][:, 0] = np.float16(np.inf)
    for mode in ("list", "fused"):
        for splits in (1, 0):
            print(f"dropped groups rows={rows} group={group} {mode} splits={splits}", flush=True)
            check(run(gpu, w, x, 0.125, mode, group, splits), ref, f"{mode} splits={splits}")


@pytest.mark.parametrize("T,K", [(9, 1024), (12, 1024), (20, 2048), (33, 1024), (300, 256)])
@pytest.mark.parametrize("rows", [1, 3])
def test_block_rows_over_xcds(gpu, T, K, rows):
    """Block-rows that do not divide by 8, with the default launch shape (33 block-rows and 3 rows: workgroups of 8
    wavefronts) and with odd numbers of workgroups per block-row."""
    M = 256 * T - 19
    w = make_weights(256 * T, K, 5200 + T)
    w = {"q_rowmajor": w["q_rowmajor"][:M].copy(), "scales": w["scales"][:M].copy()}
    x = make_x(K, "laplace", 5201, batch=rows)
    thr = quantile_threshold(x, 0.5)
    sparse = oracle.gemv(w["q_rowmajor"], w["scales"], x, thr)
    dense = oracle.gemv(w["q_rowmajor"], w["scales"], x, 0.0)
    for splits in (0, 3, 5):
        for mode in ("list", "fused", "dense"):
            print(f"block-rows T={T} K={K} rows={rows} splits={splits} {mode}", flush=True)
            check(run(gpu, w, x, thr, mode, splits=splits), dense if mode == "dense" else sparse, f"splits={splits} {mode}")


@pytest.mark.parametrize("rows", [1, 4])
def test_rounding_of_the_sums(gpu, rows):
    """SiLU products (many small activations beside few large ones) through all 28672 columns: the matrix cores round
    products down relative to the largest one.  32 products summed with 2^-24 of the largest lost per product, codes one
    to five bits below their exponent field, biased: below 2e-5 of the result in the 2-norm."""
    M, K = 256, 28672
    w = make_weights(M, K, 5300)
    r = np.random.default_rng(5301)
    g, u = r.standard_normal((2, rows, K))
    x = (g / (1 + np.exp(-g)) * u).astype(np.float16)
    q = w["q_rowmajor"]
    codes = np.stack([q & 15, q >> 4], -1).reshape(M, K).astype(np.int64)
    codes = np.where(codes > 7, codes - 16, codes)
    W = codes * np.repeat(w["scales"].view(np.float16).astype(np.float64), 128, axis=1)
    ref = x.astype(np.float64) @ W.T
    got = run(gpu, w, x, 0.0, "dense").astype(np.float64)
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"rounding rows={rows}: {rel:.2e}", flush=True)
    assert rel < 2e-5


@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("order", ["reversed", "shuffled"])
def test_full_list_in_any_order(gpu, rows, order):
    """A list of all K columns that is not ascending, slices of several passes: every column counts exactly once."""
    torch, spqt, dev = gpu
    M, K = 256, 2048
    w = make_weights(M, K, 5400)
    x_np = make_x(K, "normal", 5401, batch=rows)
    ref = oracle.gemv(w["q_rowmajor"], w["scales"], x_np, 0.0)
    cols = np.arange(K)[::-1] if order == "reversed" else np.random.default_rng(5402).permutation(K)
    packed = torch.from_numpy(spqt.spqt_pack(w["q_rowmajor"], w["scales"])).to(dev)
    x = torch.from_numpy(x_np if rows > 1 else x_np[0].copy()).to(dev)
    idx = torch.from_numpy(np.ascontiguousarray(cols, dtype=np.int32)).to(dev)
    cnt = torch.full((1,), K, dtype=torch.int32, device=dev)
    ws = spqt.new_workspace(M, K, rows)
    for splits in (1, 3, 0):
        print(f"full list {order} rows={rows} splits={splits}", flush=True)
        y = torch.full((rows, M) if rows > 1 else (M,), float("nan"), dtype=torch.float32, device=dev)
        spqt.spqt_gemv(packed, M, K, x, idx, cnt, y, ws, splits=splits)
        torch.cuda.synchronize()
        check(y.cpu().numpy().reshape(rows, M), ref, f"full list {order} splits={splits}")


@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("dist", ["laplace", "silu_product"])
def test_no_bias_is_left_in_the_sums(gpu, rows, dist):
    """The matrix cores round products down; every other pass computes with -x, so the bias cancels.  Against 64-bit
    arithmetic on 1024 x 28672, all modes: 1.0e-6 of the result at most, and 2.1e-6 to 1.3e-5 without the negation wherever there
    is a bias (not with one row at 50 %: the kept x are of like size).  The bound lies between."""
    M, K = 1024, 28672
    w = make_weights(M, K, 5500)
    r = np.random.default_rng(5501)
    if dist == "laplace":
        x = r.laplace(size=(rows, K)).astype(np.float16)
    else:
        g, u = r.standard_normal((2, rows, K))
        x = (g / (1 + np.exp(-g)) * u).astype(np.float16)
    thr = quantile_threshold(x, 0.5)
    q = w["q_rowmajor"]
    codes = np.stack([q & 15, q >> 4], -1).reshape(M, K).astype(np.int64)
    W = np.where(codes > 7, codes - 16, codes) * np.repeat(w["scales"].view(np.float16).astype(np.float64), 128, axis=1)
    kept = (np.abs(x.astype(np.float32)) >= np.float32(thr)).any(axis=0)
    for mode in ("dense", "list", "fused"):
        xs = x.astype(np.float64)
        ref = (xs if mode == "dense" else xs * kept) @ W.T
        got = run(gpu, w, x, thr, mode).astype(np.float64)
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"bias rows={rows} {dist} {mode}: {rel:.2e}", flush=True)
        assert rel < 2e-6


@pytest.mark.parametrize("rows,dist,high,low", [(1, "laplace", 1.2e-7, 3e-7), (2, "laplace", 1.2e-7, 3e-7), (4, "laplace", 1.2e-7, 3e-7),
                                                (1, "silu_product", 1.6e-7, 8e-7)])
def test_error_of_every_row_class(gpu, rows, dist, high, low):
    """The four codes of 16 bits are multiplied at different bits of their halves, so rows differ by their number modulo 4.  The matrix cores keep 24 bits below
    the largest exponent field of a product: codes 1 and 3 fill the bits below theirs, which leaves what 32-bit sums leave (1.0e-7), codes 0 and 2 sit
    four bits lower and lose up to four bits of the small x (2.1e-7; SiLU products, with more small x, 5.0e-7).  The bounds lie below what rows 1, 2 and 3 were off
    by with codes at bits 6, 4, 2 and 6 and the bias at 2 (1.2e-7 to 1.7e-7 and 3.6e-7 to 6.9e-7; SiLU products 8.3e-7 and 2.8e-6)."""
    M, K = 1024, 5120
    w = make_weights(M, K, 5600)
    r = np.random.default_rng(5601)
    if dist == "laplace":
        x = r.laplace(size=(rows, K)).astype(np.float16)
    else:
        g, u = r.standard_normal((2, rows, K))
        x = (g / (1 + np.exp(-g)) * u).astype(np.float16)
    q = w["q_rowmajor"]
    codes = np.stack([q & 15, q >> 4], -1).reshape(M, K).astype(np.int64)
    W = np.where(codes > 7, codes - 16, codes) * np.repeat(w["scales"].view(np.float16).astype(np.float64), 128, axis=1)
    ref = x.astype(np.float64) @ W.T
    off = run(gpu, w, x, 0.0, "dense").astype(np.float64) - ref
    rel = [float(np.linalg.norm(off[:, i::4]) / np.linalg.norm(ref[:, i::4])) for i in range(4)]
    print(f"error by row rows={rows} {dist}: " + " ".join(f"{v:.2e}" for v in rel), flush=True)
    assert max(rel[1], rel[3]) < high and max(rel[0], rel[2]) < low, rel


@pytest.mark.parametrize("mode", ["list", "fused", "even"])
def test_infinite_scale_in_a_pass_of_few_groups(gpu, mode):
    """A pass with fewer groups than it could take applies the scales of its last one in their place, to sums that are zero: where an earlier group's scale
    is infinite, the row's output is infinite and not NaN.  One wavefront, so that the groups share a pass; rows of every class modulo 4."""
    torch, spqt, dev = gpu
    M, K = 256, 512
    w = make_weights(M, K, 5650)
    w["q_rowmajor"][:] = 0x33
    rows = np.array([0, 1, 2, 3, 129, 255])
    for kept in ([5, 9, 130], [5, 130, 131, 200, 201], [0, 100, 127, 255]):
        x = np.zeros(K, dtype=np.float16)
        x[kept] = 1.5
        ref = oracle.gemv(w["q_rowmajor"], w["scales"], x[None], 0.5)[0]
        scales = w["scales"].copy()
        scales[rows, 0] = np.float16(np.inf)
        packed = torch.from_numpy(spqt.spqt_pack(w["q_rowmajor"], scales)).to(dev)
        xd = torch.from_numpy(x).to(dev)
        y = torch.full((M,), float("nan"), dtype=torch.float32, device=dev)
        ws = spqt.new_workspace(M, K)
        print(f"infinite scale {mode} kept={kept}", flush=True)
        if mode == "list":
            idx = torch.zeros(K, dtype=torch.int32, device=dev)
            cnt = torch.zeros(1, dtype=torch.int32, device=dev)
            spqt.spqt_gather(xd, 0.5, idx, cnt)
            spqt.spqt_gemv(packed, M, K, xd, idx, cnt, y, ws, splits=1, waves=1)
        else:
            spqt.spqt_gemv_fused(packed, M, K, xd, 0.5, y, ws, splits=1, waves=1, flags=spqt.binding.CFG_EVEN_SHARES if mode == "even" else 0)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        ref[rows] = np.inf
        assert np.all(np.isinf(got[rows]) & (got[rows] > 0)), got[rows]
        others = np.setdiff1d(np.arange(M), rows)
        check(got[others], ref[others], f"{mode} {kept}")
