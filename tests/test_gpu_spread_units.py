"""One launch, one activation row, long slices: a wavefront's columns are taken from two or four equal parts of K
(spread_of in gemv.hip).  Every column has to count exactly once, whatever the parts and the remainder of the slices:
against the oracle, |y_gpu - y_ref| <= 1e-2 + 2e-3 * |y_ref|, with kept columns that crowd into one part of K."""
import numpy as np
import pytest

import oracle
from workloads import make_weights, make_x, quantile_threshold

pytestmark = pytest.mark.gpu

# (K, workgroups per block-row): four parts with even and uneven slices, two parts with even and uneven ones, one part on both sides of the rule
SHAPES = [(2048, 1), (8960, 3), (1280, 1), (1536, 1), (2944, 1), (2176, 1), (1152, 1), (4096, 4), (32768, 2)]


def spread_of(units, parts):
    if units >= 5 * parts:
        for f in (4, 2):
            if units % f == 0 and f * -(-(units // f) // parts) <= -(-units // parts):
                return f
    return 1


def test_the_shapes_reach_every_kernel():
    assert {spread_of(K // 64, 4 * S) for K, S in SHAPES} == {1, 2, 4}


@pytest.mark.parametrize("K,splits", SHAPES)
def test_columns_from_several_parts_of_k(K, splits):
    import torch
    import paper_2511_04477_amd as spqt
    dev = torch.device("cuda:0")
    M = 300
    full = make_weights(512, K, 5600 + K)
    w = {"q_rowmajor": np.ascontiguousarray(full["q_rowmajor"][:M]), "scales": np.ascontiguousarray(full["scales"][:M])}
    packed = torch.from_numpy(spqt.spqt_pack(w["q_rowmajor"], w["scales"])).to(dev)
    ws = spqt.new_workspace(M, K)
    for dist in ("laplace", "laplace_clustered"):
        x_np = make_x(K, dist, 5601 + K)
        x = torch.from_numpy(x_np[0].copy()).to(dev)
        for sparsity in (0.0, 0.5, 0.97):
            thr = quantile_threshold(x_np, sparsity) if sparsity else 0.0
            print(f"K={K} splits={splits} parts={spread_of(K // 64, 4 * splits)} {dist} sparsity={sparsity}", flush=True)
            y = torch.full((M,), float("nan"), dtype=torch.float32, device=dev)
            spqt.spqt_gemv_fused(packed, M, K, x, thr, y, ws, splits=splits)
            torch.cuda.synchronize()
            ref = oracle.gemv(w["q_rowmajor"], w["scales"], x_np, thr)[0]
            err = np.abs(y.cpu().numpy().astype(np.float64) - ref)
            assert (err <= 1e-2 + 2e-3 * np.abs(ref)).all(), float(err.max())
