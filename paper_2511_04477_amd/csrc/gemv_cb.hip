// spqt_cb_gemv: batch-1 GEMV over the column-block variant of the zigzag layout, reading only
// the kept columns.
//
// Paper Section 4.1.2: the quantization groups run along a column (a superblock is 256
// consecutive rows of one column, in blocks of 32), so a skipped activation entry skips whole
// superblocks together with their scales; Section 4.2.2: one superblock row = 256 outputs is
// shared by n1 threadgroups x n2 simdgroups that keep partial sums locally and combine them
// once; Section 4.2.3: the compacted index list is split evenly over them.
//
// Mapping onto gfx950 (wave64), same skeleton as gemv.hip:
//   - lane (cg, seg) = (lane/8, lane%8) of a step reads bytes [16 seg, 16 seg + 16) of column cg
//     of the step: the 32 rows of ONE quantization block.  The block's scale is therefore a
//     per-lane scalar, and it is folded into the activation before the multiply:
//     acc[row] += n * (x * s) with the stored code n taken as an fp16 subnormal.
//   - a pass is simply the next (up to) 64 entries of the wavefront's slice of the index list:
//     there is no group structure to respect, no per-group fold, no flush.  The lane that owns
//     entry l loads x and the 8 scales of its column (one 16-byte load) and stages the 8
//     products in LDS; a lane picks up the product of its own (column, block) per step.
//   - the 32 accumulators run through the whole slice; the 8 column-lanes are folded once at
//     the end, and the offset-binary bias (stored = q + 8) is removed there as -8 * (sum of
//     x * s of the lane's block) over the passes whose products carry it.  With a list, and dense,
//     those of a slice's first pass, and of the second one in long slices, do not (`centre`).
//   - (Scaling x by 2^24 and by 1/16 for the odd nibbles where it is staged and read, and 64-bit addresses, took 20 of 520 instructions a pass more: list at
//     50 % with the gather 4096 x 4096 7.78 / 7.68 us, 5120 x 13824 10.5 / 10.4, K-quant in one launch at 40 % 5120 x 13824 8.96 / 8.86.)
//   - one buffer of weights refilled half by half, unpredicated clamped loads, reduction through LDS and the
//     workspace exactly as in gemv_list.hip.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kept_ring.hpp"
#include "spqt_colblock.h"

namespace {

using namespace spqt;

constexpr int kCbScaleBytes = kGroup * 16;                 // 128 columns x 8 fp16 scales
constexpr int kCbChunkBytes = SPQT_CB_CHUNK_BYTES;
static_assert(kCbChunkBytes == kCbScaleBytes + kGroup * kColBytes, "chunk size");

constexpr int kLongSlicesBit = 1 << 26;        // in the kernel's M argument, above M: see `centre`

// FUSED: the kernel applies the sparsity test itself instead of reading an index list (as
// spqt_gemv_fused does for the group layout): a wavefront's slice is a static range of columns, and its
// entries come from a ring of kept columns in LDS (kept_ring.hpp).
// BATCH activation rows share the (union) index list and ONE pass over the weights; every row has
// its own staged products, accumulators and bias sum.
//
// KQ: the K-quant flavour of the format (Section 4.1.1): the 16 header bytes of a column hold two
// fp16 superblock scales d, dmin and eight 6-bit block scales and minima; a weight is
// (d * sc_b) * q - dmin * m_b with a plain code q in 0..15.  The owner of a list entry decodes the
// header into the 8 effective scales and the 8 effective minima of its column, both times x; the
// multiply is unchanged, and the minima take the place of the offset-binary bias.
template <int WAVES, bool DENSE, bool FUSED, int BATCH, bool KQ = false>
__global__ __launch_bounds__(WAVES * 64) void spqt_cb_gemv_kernel(
    int S, int T, int K, int M, uint32_t inv, float thr, const int32_t *__restrict__ count, const int32_t *__restrict__ idx,
    const uint8_t *__restrict__ packed, const uint16_t *__restrict__ x, float *__restrict__ y, uint32_t *ws) {
    // One staging area per wavefront is enough: offsets are written and read back inside a HEAD, and the products of a pass are read
    // before those of the next one are staged.
    __shared__ uint32_t stage_off[WAVES][kPassCols];                               // byte offset of each column
    __shared__ __attribute__((aligned(16))) float stage_xs[WAVES][BATCH][kPassCols][8];  // x * scale per block
    __shared__ __attribute__((aligned(16))) float stage_xm[KQ ? WAVES : 1][BATCH][KQ ? kPassCols : 1][8];  // x * minimum
    __shared__ __attribute__((aligned(16))) float red[WAVES][BATCH][kTileRows];
    __shared__ u32x2 ring_slots[FUSED ? WAVES : 1][FUSED ? kRingSlots : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = lane >> 3;
    const int seg = lane & 7;
    const int cgr = ((cg & 1) << 2) | (cg & 2) | (cg >> 2);
    const uint32_t seg16 = (uint32_t)seg * 16u;
    const int n_raw = FUSED || DENSE ? K : *count;     // requested first
    int t, s;
    if (!block_of<WAVES>(blockIdx.x, S, T, inv, t, s)) return;
    Outputs<BATCH * kTileRows> outputs(t, s, S, T, ws, y, M);

    // (a count outside 0..K cannot come from spqt_gather; clamping keeps a corrupt one inside idx)
    const int n_ns = n_raw < 0 ? 0 : (n_raw > K ? K : n_raw);
    const int parts = S * WAVES;
    const int part = s * WAVES + wave;
    const Share share = share_of<WAVES>(n_ns, part, parts, inv);
    int pos = share.begin;
    const int end = share.end;

    const uint8_t *row_base = packed + (size_t)t * (size_t)(K >> 7) * kCbChunkBytes;

    float acc[BATCH][32];   // this lane's 32 rows, summed over its columns of the whole slice
    float bsum[BATCH];      // sum of the staged products this lane multiplied with (its block)
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        bsum[b] = 0.0f;
#pragma unroll
        for (int i = 0; i < 32; ++i) acc[b][i] = 0.0f;
    }

    constexpr float kBias = KQ ? 1.0f : 8.0f;      // what a product carries of the staged value that bsum sums
    if (pos < end) {
        KeptRing ring(ring_slots[FUSED ? wave : 0], x, K, pos, end, thr, lane);
        // Atomic loads (the same instructions): the compiler moves plain ones down to the use of their values, behind the
        // weights, and then waits for those too (10240 x 18944, list, 4 rows: 42.4 us with plain loads, 39.0 with these).
        auto fetch_k = [&](int p) -> int {
            const int e = p + lane;
            if (DENSE) return e < end ? e : 0;
            return __hip_atomic_load(element(idx, (uint32_t)(e < end ? e : end - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        };

        // One buffer of weights, refilled half by half as a pass is multiplied: when the products of steps u < 4 are done, their
        // registers receive the same steps of the next pass, whose HEAD has run before the products.  Only the last pass of a
        // list has fewer than 64 entries, so only behind the loop are steps left out.  (Two buffers with steps left out in every
        // pass: 30 registers more, and as the compiler cannot know which loads such steps left in flight it waited for all loads
        // at every other pass.  Before: list at 50 % / dense 28672 x 8192 17.8 / 26.8 us, now 16.5 / 25.0; 4096 x 14336
        // 8.8 / 11.0, now 7.8 / 10.0; 4096 x 4096 5.5 / 6.1, now 5.2 / 5.9.)
        u32x4 w[8];
        u32x4 sv;                  // raw scales and x of the entry this lane owns, of the pass whose products come next
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
            const uint32_t chunk_off = (uint32_t)(kc >> 7) * (uint32_t)kCbChunkBytes;
            const uint32_t col = (uint32_t)(kc & (kGroup - 1));
#pragma unroll
            for (int b = 0; b < BATCH; ++b) xr[b] = FUSED ? kept_x : (uint32_t)*element(x, (uint32_t)(b * K + kc));
            sv = *reinterpret_cast<const u32x4 *>(row_base + (size_t)(chunk_off + col * 16u));
            stage_off[wave][lane] = chunk_off + (uint32_t)kCbScaleBytes + col * (uint32_t)kColBytes;
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
        // The lane that owns an entry stages the 8 products x * s_b of its column, per row.
        auto stage = [&]() {
            float sc[8], mn[8];
            if (FUSED && lane >= n) sv = u32x4{0u, 0u, 0u, 0u};      // an empty pass points at column 0, which may be dropped
            if (KQ) {
                const float d = half_bits_to_float(sv.x & 0xFFFFu), dm = lane < n ? half_bits_to_float(sv.x >> 16) : 0.0f;
                const uint64_t lo = (uint64_t)sv.y | ((uint64_t)sv.z << 32);
                const uint32_t hi = sv.w;
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const int ps = 6 * b, pm = 48 + 6 * b;      // compile-time bit positions
                    const uint32_t fs = (uint32_t)(lo >> ps) & 63u;
                    uint32_t fm;
                    if (pm + 6 <= 64) fm = (uint32_t)(lo >> pm) & 63u;
                    else if (pm >= 64) fm = (hi >> (pm - 64)) & 63u;
                    else fm = ((uint32_t)(lo >> pm) | (hi << (64 - pm))) & 63u;
                    sc[b] = d * (float)fs;
                    mn[b] = dm * (float)fm;
                }
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const float xf = lane < n ? half_bits_to_float(xr[b]) : 0.0f;
                f32x4 *dst = reinterpret_cast<f32x4 *>(stage_xs[wave][b][lane]);
                if (KQ) {
                    dst[0] = f32x4{xf * sc[0], xf * sc[1], xf * sc[2], xf * sc[3]};
                    dst[1] = f32x4{xf * sc[4], xf * sc[5], xf * sc[6], xf * sc[7]};
                    f32x4 *dm4 = reinterpret_cast<f32x4 *>(stage_xm[wave][b][lane]);
                    dm4[0] = f32x4{xf * mn[0], xf * mn[1], xf * mn[2], xf * mn[3]};
                    dm4[1] = f32x4{xf * mn[4], xf * mn[5], xf * mn[6], xf * mn[7]};
                } else {
                    // (as sums with 0: the half then needs no instruction of its own to become a float)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const f16x2 h01 = as_f16x2(i ? sv.z : sv.x), h23 = as_f16x2(i ? sv.w : sv.y);
                        dst[i] = f32x4{__builtin_fmaf((float)h01.x, xf, 0.0f), __builtin_fmaf((float)h01.y, xf, 0.0f),
                                       __builtin_fmaf((float)h23.x, xf, 0.0f), __builtin_fmaf((float)h23.y, xf, 0.0f)};
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();
        };
        // Step u: 8 columns.  The bias sum takes the product itself, or x * minimum in one launch.
        auto step = [&](int u) {
            if (BATCH > 2) keep_order();     // x of several steps at once would not fit the registers
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const float xl = stage_xs[wave][b][u * 8 + cg][seg];
                fma_step(w[u], xl, acc[b]);
                if (!KQ || FUSED) bsum[b] += KQ ? stage_xm[wave][b][u * 8 + cg][seg] : xl;
            }
        };
        if (FUSED) {
            ring.fetch();
            pos = 0;                 // from here on a position among the kept columns of the slice
        } else {
            k_next = fetch_k(pos);
        }
        auto more = [&](int p) { return FUSED ? ring.more(p) : p < end; };
        const int second_end = pos + 2 * kPassCols;      // of the second pass, where it is full
        pos = head(pos);
        load_half(0);
        load_half(1);
        outputs.read_now();
        // With a list, and dense, the sums start at the bias of the first pass, so that this pass's products carry none: products of codes that are not centred
        // make sums that are further off.  Error against 64-bit arithmetic, without / with, and time (us):
        //   list, one row    14336 x 4096 at 50 %, S = 4   2.09e-7 / 1.63e-7   9.48 / 9.40
        //   dense, one row   14336 x 4096                  2.84e-7 / 2.36e-7   8.62 / 8.62     4096 x 14336   2.73e-7 / 2.28e-7   9.18 / 9.25
        //   list, 4 rows     14336 x 4096 at 60 %          2.64e-7 / 2.20e-7   18.75 / 18.76
        //   dense, 4 rows    4096 x 4096                   1.95e-7 / 1.48e-7   9.37 / 9.36
        //   K-quant          14336 x 4096 at 50 %          1.24e-7 / 1.15e-7   9.95 / 9.88     4 rows at 60 %   1.36e-7 / 1.33e-7   19.9 / 19.95
        // In one launch it is slower (K-quant 13824 x 5120 9.03 / 9.12), and the sums stay as they were.
        // Where colblock4_list_splits chose the launch shape (kLongSlicesBit), a slice well over two passes long takes the second pass so, too: where most columns are
        // kept, its four passes would be further off than the two of the slices that they replace (14336 x 4096 with S = 9, no pass centred / S = 4, one pass / S = 4,
        // two passes: all kept 2.18e-7 / 2.36e-7 / 2.00e-7, 80 % kept 2.00e-7 / 2.10e-7 / 1.75e-7; 12.8 / 11.65 / 11.71 us and 11.4 / 10.6 / 10.65).
        constexpr bool kCentred = !FUSED;
        constexpr bool kTwice = BATCH == 1 && !DENSE && !FUSED && !KQ;
        // The products of the staged pass carry no bias: the sums are ahead of it by what its x adds up to.  (K-quant: the minima of such a pass are not counted
        // at all, those of the others where the pass is staged.  Counted by the steps of every pass and taken off for this one an infinite minimum would be NaN, and the
        // steps' reads took as long or longer: list at 60 % 11008 x 4096 2 rows 11.45 / 11.29 us, 4096 x 4096 4 rows 12.62 / 12.35, dense 4096 x 4096 3 rows 8.70 / 8.42.)
        auto centre = [&](bool first_pass) {
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                float total = 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) total += KQ ? stage_xm[wave][b][u * 8 + cg][seg] : stage_xs[wave][b][u * 8 + cg][seg];
                const float even = total * (-kBias / kTwo24), odd = total * (-kBias * 16.0f / kTwo24);
                if (!KQ) bsum[b] = first_pass ? -total : bsum[b] - total;
#pragma unroll
                for (int i = 0; i < 32; ++i) acc[b][i] = first_pass ? (i & 1 ? odd : even) : acc[b][i] + (i & 1 ? odd : even);
            }
        };
        auto count_minima = [&]() {
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                if (BATCH > 2) keep_order();
#pragma unroll
                for (int u = 0; u < 8; ++u) bsum[b] += stage_xm[wave][b][u * 8 + cg][seg];
            }
        };
        if constexpr (kCentred) {
            stage();
            centre(true);
        }
        while (more(pos)) {
            if (!kCentred) stage();
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
            if (kCentred) stage();
            if (KQ && kCentred) count_minima();
            if (kTwice && pos == second_end && end - pos > kPassCols / 2 && (M & kLongSlicesBit)) centre(false);
        }
        if (!kCentred) stage();
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (u * 8 < n) step(u);
    } else {
        outputs.read_now();
    }

    // fold the 8 column-lanes once, bring the sums to true units and remove the bias
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        float r4[4];
        fold_columns(acc[b], r4);
        const float bias = sum_over_columns(bsum[b]) * kBias;
        reinterpret_cast<f32x4 *>(red[wave][b])[8 * seg + cgr] = true_rows(r4, bias);
    }
    __syncthreads();
    combine_block_row<WAVES, BATCH>(&red[0][0][0], tid, outputs);
}

template <int WAVES, int BATCH>
hipError_t launch_cb_batch(int mode, int grid, hipStream_t stream, const uint8_t *packed, const uint16_t *x,
                           const int32_t *idx, const int32_t *count, float *y, uint32_t *ws,
                           int K, int S, int T, int M, int y_half) {
    const dim3 g(grid), b(WAVES * 64);
    if (mode == 3)        // K-quant flavour, index list
        hipLaunchKernelGGL((spqt_cb_gemv_kernel<WAVES, false, false, BATCH, true>), g, b, 0, stream, S, T, K,
                           M | (y_half ? kHalfOutputBit : 0), inverse_of(S * WAVES), 0.0f, count, idx, packed, x, y, ws);
    else if (mode == 4)   // K-quant flavour, dense
        hipLaunchKernelGGL((spqt_cb_gemv_kernel<WAVES, true, false, BATCH, true>), g, b, 0, stream, S, T, K,
                           M | (y_half ? kHalfOutputBit : 0), inverse_of(S * WAVES), 0.0f, count, idx, packed, x, y, ws);
    else if (mode == 0)   // index list
        hipLaunchKernelGGL((spqt_cb_gemv_kernel<WAVES, false, false, BATCH>), g, b, 0, stream, S, T, K,
                           M | (y_half ? kHalfOutputBit : 0), inverse_of(S * WAVES), 0.0f, count, idx, packed, x, y, ws);
    else                  // dense
        hipLaunchKernelGGL((spqt_cb_gemv_kernel<WAVES, true, false, BATCH>), g, b, 0, stream, S, T, K,
                           M | (y_half ? kHalfOutputBit : 0), inverse_of(S * WAVES), 0.0f, count, idx, packed, x, y, ws);
    return hipGetLastError();
}

template <int WAVES>
hipError_t launch_cb(int mode, int batch, int grid, hipStream_t stream, const uint8_t *packed, const uint16_t *x,
                     const int32_t *idx, const int32_t *count, float *y, uint32_t *ws,
                     int K, int S, int T, int M, float thr, int y_half) {
    if (mode == 5) {      // K-quant flavour, threshold inside the kernel (batch 1)
        hipLaunchKernelGGL((spqt_cb_gemv_kernel<WAVES, false, true, 1, true>), dim3(grid), dim3(WAVES * 64), 0, stream, S, T,
                           K, M | (y_half ? kHalfOutputBit : 0), inverse_of(S * WAVES), thr, count, idx, packed, x, y, ws);
        return hipGetLastError();
    }
    if (mode == 2) {      // threshold inside the kernel (batch 1)
        hipLaunchKernelGGL((spqt_cb_gemv_kernel<WAVES, false, true, 1>), dim3(grid), dim3(WAVES * 64), 0, stream, S, T,
                           K, M | (y_half ? kHalfOutputBit : 0), inverse_of(S * WAVES), thr, count, idx, packed, x, y, ws);
        return hipGetLastError();
    }
    switch (batch) {
        case 1: return launch_cb_batch<WAVES, 1>(mode, grid, stream, packed, x, idx, count, y, ws, K, S, T, M, y_half);
        case 2: return launch_cb_batch<WAVES, 2>(mode, grid, stream, packed, x, idx, count, y, ws, K, S, T, M, y_half);
        case 3: return launch_cb_batch<WAVES, 3>(mode, grid, stream, packed, x, idx, count, y, ws, K, S, T, M, y_half);
        default: return launch_cb_batch<WAVES, 4>(mode, grid, stream, packed, x, idx, count, y, ws, K, S, T, M, y_half);
    }
}

int run_cb(int mode, int batch, const void *packed_dev, int64_t M, int64_t K, const void *x_dev, const int32_t *idx_dev,
           const int32_t *count_dev, float threshold, void *y_dev, void *workspace_dev, size_t workspace_bytes,
           void *stream, const spqt_launch_cfg *cfg) {
    if (!packed_dev || !x_dev || !y_dev) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, kGroup)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    if (cfg && (cfg->flags & ~SPQT_CFG_Y_FP16)) return SPQT_EINVAL;
    const int y_half = cfg && (cfg->flags & SPQT_CFG_Y_FP16) ? 1 : 0;
    if ((uintptr_t)packed_dev % 128 != 0 || (uintptr_t)x_dev % 2 != 0 || (uintptr_t)y_dev % (y_half ? 2 : 4) != 0)
        return SPQT_EALIGN;
    spqt_launch_cfg c;
    const Columns from = mode == 1 || mode == 4 ? Columns::dense : mode == 2 || mode == 5 ? Columns::units : Columns::list;
    c.splits = colblock_splits(tiles(M), K, from, batch, colblock4_depth(tiles(M), from, batch, mode >= 3));
    int long_slices = 0;
    if (mode == 0 && batch == 1) {
        const int few = colblock4_list_splits(tiles(M), K, c.splits);
        if (few < c.splits && !(cfg && (cfg->splits || cfg->waves))) long_slices = kLongSlicesBit;
        c.splits = few;
    }
    while (c.splits > K / kGroup) --c.splits;      // at least a quarter of a chunk per wavefront
    c.waves = 4;
    size_t need = 0;
    spqt_workspace_bytes(M, K, batch, &need);
    // (the one-launch kernel's limit is the same for matrices of any size)
    const size_t code_bytes = from == Columns::units ? 0 : (size_t)M * (size_t)K / 2;
    if (!usable_workspace(workspace_dev, workspace_bytes, need) && runs_without_workspace(tiles(M), code_bytes, from, batch)) c.splits = 1;
    if (cfg) {
        if (cfg->splits) c.splits = cfg->splits;
        if (cfg->waves) c.waves = cfg->waves;
    }
    if (c.splits < 1 || c.splits > SPQT_MAX_SPLITS) return SPQT_EINVAL;
    if (c.waves != 1 && c.waves != 2 && c.waves != 4) return SPQT_EINVAL;
    uint32_t *ws = nullptr;
    if (c.splits > 1) {
        if (!workspace_dev) return SPQT_EINVAL;
        if (workspace_bytes < need) return SPQT_ESIZE;
        if ((uintptr_t)workspace_dev % 256 != 0) return SPQT_EALIGN;
        ws = (uint32_t *)workspace_dev;
    }
    const int T = (int)tiles(M);
    const int grid = grid_blocks(T, c.splits);
    hipStream_t st = (hipStream_t)stream;
    const uint8_t *pk = (const uint8_t *)packed_dev;
    const uint16_t *xp = (const uint16_t *)x_dev;
    hipError_t err;
    switch (c.waves) {
        case 1: err = launch_cb<1>(mode, batch, grid, st, pk, xp, idx_dev, count_dev, (float *)y_dev, ws, (int)K, c.splits, T, (int)M, threshold, y_half); break;
        case 2: err = launch_cb<2>(mode, batch, grid, st, pk, xp, idx_dev, count_dev, (float *)y_dev, ws, (int)K, c.splits, T, (int)M, threshold, y_half); break;
        default: err = launch_cb<4>(mode, batch, grid, st, pk, xp, idx_dev, count_dev, (float *)y_dev, ws, (int)K, c.splits, T, (int)M | long_slices, threshold, y_half); break;
    }
    return err == hipSuccess ? SPQT_OK : SPQT_EHIP;
}

}  // namespace

extern "C" int spqt_cb_gemv(const void *packed_dev, int64_t M, int64_t K, const void *x_dev, int batch,
                            const int32_t *idx_dev, const int32_t *count_dev, void *y_dev,
                            void *workspace_dev, size_t workspace_bytes, void *stream,
                            const spqt_launch_cfg *cfg) {
    if (idx_dev && !count_dev) return SPQT_EINVAL;
    return run_cb(idx_dev ? 0 : 1, batch, packed_dev, M, K, x_dev, idx_dev, count_dev, 0.0f, y_dev, workspace_dev,
                  workspace_bytes, stream, cfg);
}

extern "C" int spqt_cb_gemv_fused(const void *packed_dev, int64_t M, int64_t K, const void *x_dev,
                                  float threshold, void *y_dev, void *workspace_dev, size_t workspace_bytes,
                                  void *stream, const spqt_launch_cfg *cfg) {
    if (threshold != threshold) return SPQT_EINVAL;
    return run_cb(2, 1, packed_dev, M, K, x_dev, nullptr, nullptr, threshold, y_dev, workspace_dev,
                  workspace_bytes, stream, cfg);
}

extern "C" int spqt_cbk_gemv_fused(const void *packed_dev, int64_t M, int64_t K, const void *x_dev,
                                   float threshold, void *y_dev, void *workspace_dev, size_t workspace_bytes,
                                   void *stream, const spqt_launch_cfg *cfg) {
    if (threshold != threshold) return SPQT_EINVAL;
    return run_cb(5, 1, packed_dev, M, K, x_dev, nullptr, nullptr, threshold, y_dev, workspace_dev,
                  workspace_bytes, stream, cfg);
}

extern "C" int spqt_cbk_gemv(const void *packed_dev, int64_t M, int64_t K, const void *x_dev, int batch,
                             const int32_t *idx_dev, const int32_t *count_dev, void *y_dev,
                             void *workspace_dev, size_t workspace_bytes, void *stream,
                             const spqt_launch_cfg *cfg) {
    if (idx_dev && !count_dev) return SPQT_EINVAL;
    return run_cb(idx_dev ? 3 : 4, batch, packed_dev, M, K, x_dev, idx_dev, count_dev, 0.0f, y_dev, workspace_dev,
                  workspace_bytes, stream, cfg);
}
