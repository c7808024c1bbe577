// The column-block GEMV for bit-widths other than 4 (gemv_cb8.hip, gemv_cb2.hip): one kernel body, the
// width-specific parts supplied by a format type F.
//
// Paper Section 4.1.3 states that the column-wise layout carries over to other bit-widths.  What the
// 4-bit kernels are built around is kept at every width: one activation column's weights of a block-row
// are ONE 128-byte run, read by 8 lanes with one 16-byte load each, 8 columns per wavefront load, 64
// list entries per pass; the height of a block-row follows from the width (128 bytes of codes).
// Everything else follows spqt_cb_gemv_kernel: even split of the index list over the S x WAVES
// wavefronts of a block-row (Section 4.2.3), the scales folded into x by the lane that owns the list
// entry, one buffer of weights refilled half by half with unpredicated clamped loads, one fold of the 8 column-lanes at
// the end, reduction through LDS and the workspace.  Three modes: list-driven, dense (every
// column, no list), and ONE-LAUNCH (FUSED, one activation row): the kernel applies the sparsity test of
// Section 2 itself on static column ranges and takes its entries from a ring of kept columns in LDS (kept_ring.hpp), so
// no index list exists.
// BATCH activation rows (Section 3.3: small beams) share the union index list and ONE pass over the
// weights; every row has its own staged products, accumulators and offset sums.
//
// A format type F provides
//   kRows, kBlocks            rows of a block-row, 32-row blocks in it (one fp16 scale each per column)
//   kScaleBytes, kChunkBytes  scale bytes per 128-column chunk (2 * kBlocks per column), chunk size
//   kAcc                      accumulators per lane (rows per lane = kRows / 8)
//   Scales                    the raw scale bytes of one column, as loaded (load_scales)
//   stage(xf, sv, dst)        dst[b] = xf * scale_b for the kBlocks blocks, by the lane that owns the entry
//   Mine                      the staged products of the block(s) a lane's rows lie in (read_mine)
//   step(w, mine, acc, bs)    one column: acc += code-fields * mine, bs += mine
//   finish(acc, bs, seg, cgr, red)   fold the 8 column-lanes, undo field weights and code offset, rows to red
#ifndef SPQT_COLBLOCK_WIDTH_HPP
#define SPQT_COLBLOCK_WIDTH_HPP

#include "kept_ring.hpp"

namespace spqt {

template <class F, int WAVES, bool DENSE, bool FUSED, int BATCH = 1>
__device__ __forceinline__ void colblock_width_gemv(int S, int T, int K, int M, uint32_t inv, float thr, const int32_t *__restrict__ count,
                                                    const int32_t *__restrict__ idx, const uint8_t *__restrict__ packed,
                                                    const uint16_t *__restrict__ x, float *__restrict__ y, uint32_t *ws) {
    __shared__ uint32_t stage_off[WAVES][kPassCols];                                          // byte offset of each column
    static_assert(!FUSED || BATCH == 1, "the one-launch mode takes one activation row");
    __shared__ __attribute__((aligned(16))) float stage_xs[WAVES][BATCH][kPassCols][F::kBlocks];   // x * scale per block
    __shared__ __attribute__((aligned(16))) float red[WAVES][BATCH][F::kRows];
    __shared__ u32x2 ring_slots[FUSED ? WAVES : 1][FUSED ? kRingSlots : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = lane >> 3;      // column of the step this lane reads
    const int seg = lane & 7;      // eighth of the block-row this lane reads
    const int cgr = ((cg & 1) << 2) | (cg & 2) | (cg >> 2);
    const uint32_t seg16 = (uint32_t)seg * 16u;
    // what is split evenly: the kept-column list, or (dense, one launch) all columns
    const int n_raw = FUSED || DENSE ? K : *count;     // requested first
    int t, s;
    if (!block_of<WAVES>(blockIdx.x, S, T, inv, t, s)) return;
    Outputs<BATCH * F::kRows> outputs(t, s, S, T, ws, y, M);

    const int n_ns = n_raw < 0 ? 0 : (n_raw > K ? K : n_raw);
    const int parts = S * WAVES;
    const int part = s * WAVES + wave;
    const Share share = share_of<WAVES>(n_ns, part, parts, inv);
    int pos = share.begin;
    const int end = share.end;

    const uint8_t *row_base = packed + (size_t)t * (size_t)(K >> 7) * F::kChunkBytes;

    float acc[BATCH][F::kAcc];
    typename F::Sums bs[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        bs[b] = F::zero_sums();
#pragma unroll
        for (int i = 0; i < F::kAcc; ++i) acc[b][i] = 0.0f;
    }

    if (pos < end) {
        KeptRing ring(ring_slots[FUSED ? wave : 0], x, K, pos, end, thr, lane);
        // atomic loads (the same instructions): plain ones the compiler moves behind the weights, to their use
        auto fetch_k = [&](int p) -> int {
            const int e = p + lane;
            if (DENSE) return e < end ? e : 0;
            return __hip_atomic_load(idx + (e < end ? e : end - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        };
        // One buffer of weights, refilled half by half as a pass is multiplied: when the products of steps u < 4 are done, their
        // registers receive the same steps of the next pass, whose HEAD has run before the products.  Only the last pass of a
        // list has fewer than 64 entries, so only behind the loop are steps left out.  (Two buffers with steps left out in every
        // pass: 30 registers more, and as the compiler cannot know which loads such steps left in flight it waited for all loads
        // at every other pass.  Before, list at 50 % / dense: 8-bit 4096 x 14336 10.2 / 14.1 us, now 9.5 / 13.3; 28672 x 8192 24.2 / 40.3, now
        // 23.5 / 39.8; 2-bit 4096 x 14336 9.8 / 12.9, now 8.7 / 11.4; 28672 x 8192 15.9 / 22.8, now 14.4 / 21.3.)
        u32x4 w[8];
        typename F::Scales sv;                  // raw scales and x of the entry this lane owns, of the pass whose products come next
        uint32_t xr[BATCH], off[8];        // off: byte offsets of the columns this lane reads
        int n, k_next = 0;                 // entries of that pass (wave-uniform); the lane's entry of the one after it

        // HEAD of the pass at list position p: request the entries of the pass after it, this pass's x and scales, and deal the
        // offsets of its columns.  Lanes past the pass point at its first column and carry x = 0.  Returns where the next pass starts.
        auto head = [&](int p) -> int {
            int kk = k_next;
            uint32_t kept_x = 0u;
            if constexpr (FUSED) {
                const u32x2 kept = ring.take(p, n);
                kk = (int)kept.x;
                kept_x = kept.y;
            } else {
                n = end - p < kPassCols ? end - p : kPassCols;
                k_next = fetch_k(p + kPassCols);
            }
            const int k_first = n ? __builtin_amdgcn_readfirstlane(kk) : 0;
            const int kc = lane < n ? kk : k_first;
            const uint32_t chunk_off = (uint32_t)(kc >> 7) * (uint32_t)F::kChunkBytes;
            const uint32_t col = (uint32_t)(kc & (kGroup - 1));
#pragma unroll
            for (int b = 0; b < BATCH; ++b) xr[b] = FUSED ? kept_x : (uint32_t)x[(size_t)b * K + kc];
            sv = F::load_scales(row_base + (size_t)(chunk_off + col * (uint32_t)(2 * F::kBlocks)));
            stage_off[wave][lane] = chunk_off + (uint32_t)F::kScaleBytes + col * (uint32_t)kColBytes;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int u = 0; u < 8; ++u) off[u] = stage_off[wave][u * 8 + cg] + seg16;
            __builtin_amdgcn_wave_barrier();
            return p + n;
        };
        auto load_half = [&](int half) {
#pragma unroll
            for (int u = 4 * half; u < 4 * half + 4; ++u)
                w[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(row_base + (size_t)off[u]));
        };
        // The lane that owns an entry stages the products x * s_b of its column; a step (8 columns) takes those of the lane's block(s).
        auto stage = [&]() {
            if (FUSED && lane >= n) sv = typename F::Scales{};     // an empty pass points at column 0, which may be dropped
#pragma unroll
            for (int b = 0; b < BATCH; ++b) F::stage(lane < n ? half_bits_to_float(xr[b]) : 0.0f, sv, stage_xs[wave][b][lane]);
            __builtin_amdgcn_wave_barrier();
        };
        auto step = [&](int u) {
            if (BATCH * F::kAcc > 64) keep_order();     // x of several steps at once would not fit the registers
#pragma unroll
            for (int b = 0; b < BATCH; ++b) F::step(w[u], F::read_mine(stage_xs[wave][b][u * 8 + cg], seg), acc[b], bs[b]);
        };
        if (FUSED) {
            ring.fetch();
            pos = 0;                 // from here on a position among the kept columns of the slice
        } else {
            k_next = fetch_k(pos);
        }
        auto more = [&](int p) { return FUSED ? ring.more(p) : p < end; };
        pos = head(pos);
        load_half(0);
        load_half(1);
        outputs.read_now();
        auto pass = [&]() {          // every pass but the last one
            stage();
            const bool whole = !FUSED || n > kPassCols / 2;
            pos = head(pos);
            keep_order();
#pragma unroll
            for (int u = 0; u < 4; ++u) step(u);
            keep_order();
            load_half(0);
            keep_order();
            if (whole) {
#pragma unroll
                for (int u = 4; u < 8; ++u) step(u);
            }
            keep_order();
            load_half(1);
            keep_order();
        };
        // Many accumulators: a slice of one pass has code of its own.  The compiler then knows that the loop runs, and keeps fewer of them in the
        // accumulator file of the matrix cores, from where each use is a copy away (2-bit, 3 rows: 287 copies in the code, not 537).  Without / with,
        // 2-bit: list at 60 % a row, 3 rows 512 x 1024 11.1 / 10.3 us, 28672 x 8192 44.9 / 39.9, 2 rows 512 x 1024 7.0 / 6.7.
        constexpr bool kAlone = BATCH * F::kAcc > 64;
        if (kAlone && !more(pos)) {
            stage();
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (u == 0 || u * 8 < n) step(u);
        } else {
            if constexpr (kAlone) {
                do pass();
                while (more(pos));
            } else {
                while (more(pos)) pass();
            }
            stage();
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (u * 8 < n) step(u);
        }
    } else {
        outputs.read_now();
    }

#pragma unroll
    for (int b = 0; b < BATCH; ++b) F::finish(acc[b], bs[b], seg, cgr, red[wave][b]);
    __syncthreads();
    combine_block_row<WAVES, BATCH, F::kRows>(&red[0][0][0], tid, outputs);
}

// Host side shared by the entry points: argument checks, launch shape, workspace, grid.  `launch` starts the
// kernel for (waves, mode) with mode 0 = index list, 1 = dense, 2 = one launch (batch 1 only).  without_workspace: the
// default shape is one workgroup per block-row if the call brings no usable workspace.
template <class F, class Launch>
int colblock_width_run(int mode, int batch, int max_splits, int default_splits, bool without_workspace, const void *packed_dev, int64_t M, int64_t K,
                       const void *x_dev, const int32_t *idx_dev, const int32_t *count_dev, void *y_dev,
                       void *workspace_dev, size_t workspace_bytes, const spqt_launch_cfg *cfg, Launch launch) {
    if (!packed_dev || !x_dev || !y_dev) return SPQT_EINVAL;
    if (mode == 0 && !count_dev) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, kGroup)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH || (mode == 2 && batch != 1)) return SPQT_ESHAPE;
    if (cfg && (cfg->flags & ~SPQT_CFG_Y_FP16)) return SPQT_EINVAL;
    const int y_half = cfg && (cfg->flags & SPQT_CFG_Y_FP16) ? 1 : 0;
    if ((uintptr_t)packed_dev % 128 != 0 || (uintptr_t)x_dev % 2 != 0 || (uintptr_t)y_dev % (y_half ? 2 : 4) != 0)
        return SPQT_EALIGN;
    const int64_t T64 = (M + F::kRows - 1) / F::kRows;
    size_t need = 0;
    spqt_workspace_bytes(M, K, batch, &need);
    int S = without_workspace && !usable_workspace(workspace_dev, workspace_bytes, need) ? 1 : default_splits;
    int waves = 4;
    if (cfg) {
        if (cfg->splits) S = cfg->splits;
        if (cfg->waves) waves = cfg->waves;
    }
    if (S < 1 || S > max_splits) return SPQT_EINVAL;
    if (waves != 1 && waves != 2 && waves != 4) return SPQT_EINVAL;
    uint32_t *ws = nullptr;
    if (S > 1) {
        if (!workspace_dev) return SPQT_EINVAL;
        if (workspace_bytes < need) return SPQT_ESIZE;
        if ((uintptr_t)workspace_dev % 256 != 0) return SPQT_EALIGN;
        ws = (uint32_t *)workspace_dev;
    }
    const int T = (int)T64;
    const int grid = grid_blocks(T, S);
    const int m_and_flags = (int)M | (y_half ? kHalfOutputBit : 0);
    const hipError_t err = launch(waves, mode, grid, ws, S, T, m_and_flags);
    return err == hipSuccess ? SPQT_OK : SPQT_EHIP;
}

}  // namespace spqt
#endif
