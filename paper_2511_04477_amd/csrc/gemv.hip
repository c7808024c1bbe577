// The GEMV in ONE launch with static column ranges (spqt_gemv_fused, spqt_gemv_fused_rows), and the host side of every
// group-layout entry point.
//
// Paper Section 2: a column is sparse iff |x_i| < threshold; Section 4.2.2 (zigzag kernel): one block-row = 256 outputs is
// shared by n1 threadgroups x n2 simdgroups that keep partial sums locally and combine them once.  Instead of reading an
// index list, the kernel tests x itself: the slice of a wavefront is a static range of columns (K split evenly over the S*WAVES
// wavefronts of the block-row, to the column or to the unit: slice_quantum).  A wavefront compacts its range, kRefill units of 64 columns at a time and only
// as its passes need them, into a ring of (column, x) entries in LDS - lane l tests the unit's column l, a ballot gives the kept
// set, mbcnt the rank - and takes its passes (pass.hpp) from the ring exactly as gemv_list.hip takes them from idx.
//
// Why a ring: with one pass per 64-column unit a pass is as full as the unit (38 of 64 slots at 40 % sparsity), and
// empty slots cost their load and multiply issue.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "pass.hpp"

namespace {

using namespace spqt;

// BATCH activation rows share one pass over the weights: a column is visited if ANY row keeps it; with the own-sets flag
// (in M) every row contributes only where it keeps the column itself (its x is staged as 0 elsewhere), which is that
// row's batch-1 result.
// COMPACT == false is an ablation: same test, same static ranges, but NO compaction - a dropped column keeps its entry
// with x = 0 (and re-reads a kept column's line), so skipping saves memory traffic but not one product.
constexpr int kRefill = 4;                   // units compacted together: their x is requested one refill ahead
// SPREAD: a slice is a static range of each of SPREAD equal parts of K, at the same place in each (spread_of below), not one range.
constexpr int kRing = 512;                   // ring entries per wavefront; a refill adds at most 256 to at most 63 live ones
template <int WAVES, int BATCH, bool COMPACT, int SPREAD>
__global__ __launch_bounds__(WAVES * 64) void spqt_gemv_fused_kernel(
    int S, int T, int K, int M, uint32_t inv, float thr, const uint16_t *__restrict__ x, const uint8_t *__restrict__ packed,
    float *__restrict__ y, uint32_t *ws) {
    constexpr int kGroups = groups_per_pass(BATCH);
    __shared__ __attribute__((aligned(16))) StagedX staged[WAVES];
    // the wavefront's kept columns: {column, x[0] | x[1] << 16}, x[2] | x[3] << 16 (+ 64 entries that nothing reads)
    __shared__ u32x2 ring[WAVES][kRing + 64];
    __shared__ uint32_t ring23[BATCH > 2 ? WAVES : 1][BATCH > 2 ? kRing + 64 : 1];
    __shared__ __attribute__((aligned(16))) float red[WAVES][BATCH][kTileRows];

    SPQT_TL_BEGIN();
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15;       // 16-row segment of the block-row this lane reads
    const uint32_t n8 = (uint32_t)n * 8u;
    const uint32_t out4 = (uint32_t)(4 * n + (lane >> 4));    // the lane's 4 outputs: rows 4 out4 .. 4 out4 + 3
    int t, s;
    if (!block_of<WAVES>(blockIdx.x, S, T, inv, t, s)) return;
    Outputs<BATCH * kTileRows> outputs(t, s, S, T, ws, y, M);

    // Positions are columns of one part of K; SPREAD columns that lie `apart` from each other share one.  A refill takes kStep
    // units of each part, and unit_at(u, i) is the first column of unit i of the refill at position u.
    constexpr int kStep = kRefill / SPREAD;
    const int apart = K / SPREAD;
    auto unit_at = [&](int at, int i) { return at + i % kStep * kPassCols + i / kStep * apart; };
    const int parts = S * WAVES;
    const int part = s * WAVES + wave;
    constexpr int kQuantum = slice_quantum(BATCH, COMPACT);
    const Share share = share_of<WAVES>(apart / kQuantum, part, parts, inv);
    int u = share.begin * kQuantum;
    const int end = share.end * kQuantum;
    SPQT_TL(1);

    // quantization groups of 128 or 64 columns
    const int log2g = M & kGroup64Bit ? 6 : 7;
    const uint32_t chunk_b = (uint32_t)(kScaleBytes + (kColBytes << log2g));
    const uint8_t *row_base = packed + (size_t)t * (size_t)(K >> log2g) * chunk_b;

    float acc[BATCH][4];   // rows 4 out4 + p of the block-row, scaled, in the products' units
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
#pragma unroll
        for (int p = 0; p < 4; ++p) acc[b][p] = 0.0f;

    if (u < end) {
        const bool own = BATCH > 1 && (M & kOwnSetsBit) != 0;
        int filled = 0;                   // entries written to the ring so far; u = the next position to compact

        // This lane's x of kRefill units from position `at` on (index clamped: values past the slice are unused).  Atomic loads (the
        // same instructions) because the compiler moves plain ones down to the use of their values, behind the weights, and
        // then waits for those too.
        uint16_t xr[kRefill][BATCH];
        auto fetch_x = [&](int at) {
#pragma unroll
            for (int i = 0; i < kRefill; ++i) {
                const int c = unit_at(at, i) + lane;
#pragma unroll
                for (int b = 0; b < BATCH; ++b)
                    xr[i][b] = __hip_atomic_load(element(x, (uint32_t)(b * K + (c < K ? c : K - 1))), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
        };

        // Compacts kRefill more units into the ring.  Dropped columns go to the entries behind the ring, which keeps the
        // code free of branches.
        auto refill = [&]() {
#pragma unroll
            for (int i = 0; i < kRefill; ++i) {
                bool kb[BATCH];
                bool keep = false;
#pragma unroll
                for (int b = 0; b < BATCH; ++b) {
                    kb[b] = u + i % kStep * kPassCols + lane < end && !(__builtin_fabsf(half_bits_to_float(xr[i][b])) < thr);
                    keep = keep || kb[b];
                }
                const uint64_t mask = __ballot(keep);
                const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                uint32_t xb[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int b = 0; b < BATCH; ++b) xb[b] = keep && (!own || kb[b]) ? (uint32_t)xr[i][b] : 0u;
                const int first = mask ? (int)__builtin_ctzll(mask) : 0;
                const bool enter = COMPACT ? keep : mask != 0ull;
                const int at = enter ? ((filled + (COMPACT ? rank : lane)) & (kRing - 1)) : kRing + lane;
                ring[wave][at] = u32x2{(uint32_t)(unit_at(u, i) + (keep ? lane : first)), xb[0] | (xb[1] << 16)};
                if (BATCH > 2) ring23[wave][at] = xb[2] | (xb[3] << 16);
                filled += COMPACT ? (int)__popcll(mask) : (mask ? kPassCols : 0);
            }
            filled = __builtin_amdgcn_readfirstlane(filled);
            u += kStep * kPassCols;
            __builtin_amdgcn_wave_barrier();
        };

        PassHead<BATCH> h;
        // HEAD of the pass that starts at entry p.  One refill at most, so a pass takes what is there (nothing, if kRefill
        // units keep nothing); the next units' x is requested every time, refilled or not, so that the number of loads in
        // flight is the same on every path.
        auto head = [&](int p) -> int {
            if (filled < p + kPassCols && u < end) refill();
            fetch_x(u);
            const int e = p + lane;
            const u32x2 v = ring[wave][e & (kRing - 1)];
            const uint32_t v23 = BATCH > 2 ? ring23[wave][e & (kRing - 1)] : 0u;
            const int kk = e < filled ? (int)v.x : -1;
            const Deal d = deal_columns<kGroups>(h, kk, log2g, chunk_b, lane);
            const uint32_t xv[4] = {v.y & 0xFFFFu, v.y >> 16, v23 & 0xFFFFu, v23 >> 16};
#pragma unroll
            for (int b = 0; b < BATCH; ++b) h.xraw[b] = (uint16_t)xv[b];
            return p + d.n;
        };
        fetch_x(u);
        run_passes<BATCH, kGroups, true, false>(staged[wave], row_base, lane, n8, out4, part, 0, h, head,
                                   [&](int p) { return p < filled || u < end; }, [&]() { outputs.read_now(); }, [&]() {}, acc);
    } else {
        outputs.read_now();
    }

    SPQT_TL(4);
    // back to true units, then the WAVES wavefronts are combined through LDS
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
        reinterpret_cast<f32x4 *>(red[wave][b])[out4] = f32x4{acc[b][0] * kUnit[0], acc[b][1] * kUnit[1], acc[b][2] * kUnit[2], acc[b][3] * kUnit[3]};
    __syncthreads();
    SPQT_TL(5);
    combine_block_row<WAVES, BATCH>(&red[0][0][0], tid, outputs);
    SPQT_TL_END(WAVES, wave, lane, S > 1 && s == S - 1);
}

SPQT_TL_SETTER(spqt_timeline_set_gemv)

__global__ void spqt_fill_zero_kernel(uint32_t *p, size_t n_words) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_words) p[i] = 0u;
}

template <int WAVES, int BATCH, bool COMPACT, int SPREAD = 1>
void start_fused(int grid, hipStream_t stream, const uint8_t *packed, const uint16_t *x, float thr, float *y, uint32_t *ws,
                 int K, int S, int T, int m_and_flags) {
    hipLaunchKernelGGL((spqt_gemv_fused_kernel<WAVES, BATCH, COMPACT, SPREAD>), dim3(grid), dim3(WAVES * 64), 0, stream, S, T, K,
                       m_and_flags, inverse_of(S * WAVES), thr, x, packed, y, ws);
}

// In how many parts of K a slice of the one-row kernel lies, with `parts` slices.  With one range per slice, activations whose kept
// columns crowd into one part of K leave the other wavefronts idle for as long as the crowded slices have passes.  28672 x 8192 at 50 %, 7 of 8
// kept columns in the first half, one range / four 22.9 / 15.8 us; evenly kept columns 17.6 / 17.4; 14336 x 14336, two ranges, 21.0 / 15.3 and
// 15.6 / 15.6.  Only where no slice gets more units to compact by it (14336 x 14336 in four parts: 16 instead of 14) and from 5 units per slice on: shorter
// slices are a pass or two either way.
inline int spread_of(int units, int parts) {
    if (units < 5 * parts) return 1;
    for (int f = 4; f > 1; f /= 2)
        if (units % f == 0 && f * ((units / f + parts - 1) / parts) <= (units + parts - 1) / parts) return f;
    return 1;
}

hipError_t launch_fused(int waves, bool compact, int grid, hipStream_t st, const uint8_t *pk, const uint16_t *x, float thr,
                        float *y, uint32_t *ws, int K, int S, int T, int mf) {
    const int spread = waves == 4 && compact ? spread_of(K / kPassCols, S * 4) : 1;
    if (spread == 4) start_fused<4, 1, true, 4>(grid, st, pk, x, thr, y, ws, K, S, T, mf);
    else if (spread == 2) start_fused<4, 1, true, 2>(grid, st, pk, x, thr, y, ws, K, S, T, mf);
    else switch (waves) {
        case 1: compact ? start_fused<1, 1, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf) : start_fused<1, 1, false>(grid, st, pk, x, thr, y, ws, K, S, T, mf); break;
        case 2: compact ? start_fused<2, 1, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf) : start_fused<2, 1, false>(grid, st, pk, x, thr, y, ws, K, S, T, mf); break;
        default: compact ? start_fused<4, 1, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf) : start_fused<4, 1, false>(grid, st, pk, x, thr, y, ws, K, S, T, mf); break;
    }
    return hipGetLastError();
}

// One launch for 2..4 activation rows (4 or 8 wavefronts per workgroup).
hipError_t launch_fused_rows(int waves, int batch, int grid, hipStream_t st, const uint8_t *pk, const uint16_t *x, float thr,
                             float *y, uint32_t *ws, int K, int S, int T, int mf) {
    switch (batch) {
        case 2: start_fused<4, 2, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf); break;
        case 3: waves == 8 ? start_fused<8, 3, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf) : start_fused<4, 3, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf); break;
        default: waves == 8 ? start_fused<8, 4, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf) : start_fused<4, 4, true>(grid, st, pk, x, thr, y, ws, K, S, T, mf); break;
    }
    return hipGetLastError();
}

}  // namespace

extern "C" int spqt_workspace_bytes(int64_t M, int64_t K, int batch, size_t *out_bytes) {
    if (!out_bytes) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, kGroup)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    *out_bytes = kWorkspaceHead + (size_t)tiles(M) * kTileRows * SPQT_MAX_SPLITS * 2 * sizeof(float) * (size_t)batch;
    return SPQT_OK;
}

extern "C" int spqt_workspace_init(void *workspace_dev, size_t workspace_bytes, void *stream) {
    if (!workspace_dev || workspace_bytes < kWorkspaceHead) return SPQT_EINVAL;
    if ((uintptr_t)workspace_dev % 256 != 0) return SPQT_EALIGN;
    // The poison flag and every exchange word start at zero: clear all of it.
    size_t words = workspace_bytes / 4;
    hipLaunchKernelGGL(spqt_fill_zero_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, (uint32_t *)workspace_dev, words);
    return hipGetLastError() == hipSuccess ? SPQT_OK : SPQT_EHIP;
}

extern "C" int spqt_default_cfg(int64_t M, int64_t K, int batch, int sparse, spqt_launch_cfg *out) {
    if (!out) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, kGroup)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    default_shape(M, K, batch, out);
    return SPQT_OK;
}

namespace {

// Bytes of workspace a call with S workgroups per block-row asks for: what spqt_workspace_bytes reports, or just the exchange
// words of this launch (`tight`).
size_t needed_bytes(int64_t M, int64_t K, int batch, int S, bool tight) {
    size_t need = 0;
    if (tight) return exchange_bytes(tiles(M), kTileRows, S, batch);
    spqt_workspace_bytes(M, K, batch, &need);
    return need;
}

// M and the flags of a call as the kernels take them.
int kernel_rows(int64_t M, int group, int y_half) { return (int)M | (y_half ? kHalfOutputBit : 0) | (group == kGroup ? 0 : kGroup64Bit); }

// spqt_gemv_ex, and the allocation-free variant: `tight` accepts a workspace that holds just the
// exchange words this launch shape touches instead of the size spqt_workspace_bytes reports.
int gemv_run(const void *packed_dev, int64_t M, int64_t K, int group, const void *x_dev, int batch,
             const int32_t *idx_dev, const int32_t *count_dev, void *y_dev, void *workspace_dev,
             size_t workspace_bytes, void *stream, const spqt_launch_cfg *cfg, bool tight) {
    if (!packed_dev || !x_dev || !y_dev) return SPQT_EINVAL;
    if (idx_dev && !count_dev) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, group)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    const int y_half = cfg && (cfg->flags & SPQT_CFG_Y_FP16) ? 1 : 0;
    if ((uintptr_t)packed_dev % 128 != 0 || (uintptr_t)x_dev % 2 != 0 || (uintptr_t)y_dev % (y_half ? 2 : 4) != 0)
        return SPQT_EALIGN;

    const bool one_group = cfg && (cfg->flags & SPQT_CFG_GROUP_PASSES);
    spqt_launch_cfg c;
    if (cfg && (cfg->splits || cfg->waves)) {
        choose_cfg(M, K, batch, &c);
        if (cfg->splits) c.splits = cfg->splits;
        if (cfg->waves) c.waves = cfg->waves;
        // 8 wavefronts per workgroup (two per SIMD) exist for 3 and 4 activation rows and for an index list with one
        if (c.waves == 8 && batch < 3 && (!idx_dev || batch > 1 || one_group)) return SPQT_EINVAL;
    } else {
        default_shape(M, K, batch, &c);
    }
    if (c.splits < 1 || c.splits > SPQT_MAX_SPLITS) return SPQT_EINVAL;
    if (c.waves != 1 && c.waves != 2 && c.waves != 4 && c.waves != 8) return SPQT_EINVAL;

    const size_t need = needed_bytes(M, K, batch, c.splits, tight);
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
    hipError_t err;
    const uint8_t *pk = (const uint8_t *)packed_dev;
    const uint16_t *xp = (const uint16_t *)x_dev;
    const ListLaunch a = {pk, xp, idx_dev, count_dev, (float *)y_dev, ws, (int)K, c.splits, T, kernel_rows(M, group, y_half)};
    err = launch_gemv_list(c.waves, batch, one_group, grid, st, a);
    if (err != hipSuccess) return SPQT_EHIP;
    return SPQT_OK;
}

// Exchange words for callers that cannot bring a workspace: one array per GPU, in the library's own
// image, zero when the image is loaded and put back to zero by every call that used it.
constexpr size_t kStaticScratchBytes = SPQT_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void *scratch_of_device[kMaxDevices];   // this process's address of `scratch` on each GPU, once known

// The array's name is only a host-side handle: its device address comes from the runtime, per GPU.
int static_scratch(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SPQT_EHIP;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_of_device[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SPQT_EHIP;
        scratch_of_device[dev] = p;
    }
    *out = scratch_of_device[dev];
    return SPQT_OK;
}

}  // namespace

extern "C" int spqt_gemv_ex(const void *packed_dev, int64_t M, int64_t K, int group, const void *x_dev,
                            int batch, const int32_t *idx_dev, const int32_t *count_dev, void *y_dev,
                            void *workspace_dev, size_t workspace_bytes, void *stream,
                            const spqt_launch_cfg *cfg) {
    return gemv_run(packed_dev, M, K, group, x_dev, batch, idx_dev, count_dev, y_dev, workspace_dev,
                    workspace_bytes, stream, cfg, false);
}

extern "C" int spqt_gemv_static(const void *packed_dev, int64_t M, int64_t K, int group, const void *x_dev,
                                int batch, const int32_t *idx_dev, const int32_t *count_dev, float *y_dev,
                                void *stream) {
    // Shape errors first, so that a bad call never touches the runtime.
    if (int rc = check_shape(M, K, group)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    spqt_launch_cfg c;
    choose_cfg(M, K, batch, &c);
    if (c.splits > 1 && exchange_bytes(tiles(M), kTileRows, c.splits, batch) > kStaticScratchBytes) return SPQT_ESIZE;
    void *ws = nullptr;
    if (int rc = static_scratch(&ws)) return rc;
    return gemv_run(packed_dev, M, K, group, x_dev, batch, idx_dev, count_dev, y_dev, ws, kStaticScratchBytes,
                    stream, nullptr, true);
}

extern "C" int spqt_gemv_fused(const void *packed_dev, int64_t M, int64_t K, int group, const void *x_dev,
                               float threshold, void *y_dev, void *workspace_dev, size_t workspace_bytes,
                               void *stream, const spqt_launch_cfg *cfg) {
    if (!packed_dev || !x_dev || !y_dev) return SPQT_EINVAL;
    if (threshold != threshold) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, group)) return rc;
    const int y_half = cfg && (cfg->flags & SPQT_CFG_Y_FP16) ? 1 : 0;
    if ((uintptr_t)packed_dev % 128 != 0 || (uintptr_t)x_dev % 2 != 0 || (uintptr_t)y_dev % (y_half ? 2 : 4) != 0)
        return SPQT_EALIGN;
    // Static column ranges by default; even shares of the kept columns (gemv_bal.hip) when the caller asks
    // for them - that kernel reads x 16 bytes at a time and holds all of it in LDS (64 KB).
    const bool even_shares = cfg && (cfg->flags & SPQT_CFG_EVEN_SHARES);
    if (even_shares && ((cfg->flags & SPQT_CFG_NO_COMPACTION) || K > 32768 || (uintptr_t)x_dev % 16 != 0)) return SPQT_EINVAL;
    const bool static_ranges = !even_shares;
    spqt_launch_cfg c;
    if (cfg && (cfg->splits || cfg->waves)) {
        choose_cfg(M, K, 1, &c);
        if (cfg->splits) c.splits = cfg->splits;
        if (cfg->waves) c.waves = cfg->waves;
    } else {
        default_shape(M, K, 1, &c);
    }
    if (c.splits < 1 || c.splits > SPQT_MAX_SPLITS) return SPQT_EINVAL;
    if (c.waves != 1 && c.waves != 2 && c.waves != 4) return SPQT_EINVAL;
    const size_t need = needed_bytes(M, K, 1, c.splits, false);
    uint32_t *ws = nullptr;
    if (c.splits > 1) {
        if (!workspace_dev) return SPQT_EINVAL;
        if (workspace_bytes < need) return SPQT_ESIZE;
        if ((uintptr_t)workspace_dev % 256 != 0) return SPQT_EALIGN;
        ws = (uint32_t *)workspace_dev;
    }
    const int T = (int)tiles(M);
    const int grid = grid_blocks(T, c.splits);
    const bool compact = !(cfg && (cfg->flags & SPQT_CFG_NO_COMPACTION));
    hipStream_t st = (hipStream_t)stream;
    const uint8_t *pk = (const uint8_t *)packed_dev;
    const uint16_t *xp = (const uint16_t *)x_dev;
    hipError_t err;
    if (!static_ranges) {
        err = launch_gemv_bal(c.waves, grid, st, pk, xp, threshold, (float *)y_dev, ws, (int)K,
                              c.splits, T, kernel_rows(M, group, y_half));
        return err == hipSuccess ? SPQT_OK : SPQT_EHIP;
    }
    err = launch_fused(c.waves, compact, grid, st, pk, xp, threshold, (float *)y_dev, ws, (int)K, c.splits, T,
                       kernel_rows(M, group, y_half));
    return err == hipSuccess ? SPQT_OK : SPQT_EHIP;
}

extern "C" int spqt_gemv_fused_rows(const void *packed_dev, int64_t M, int64_t K, int group, const void *x_dev, int batch,
                                    float threshold, int own_sets, void *y_dev, void *workspace_dev,
                                    size_t workspace_bytes, void *stream, const spqt_launch_cfg *cfg) {
    if (batch == 1) return spqt_gemv_fused(packed_dev, M, K, group, x_dev, threshold, y_dev, workspace_dev, workspace_bytes, stream, cfg);
    if (!packed_dev || !x_dev || !y_dev) return SPQT_EINVAL;
    if (threshold != threshold) return SPQT_EINVAL;
    if (int rc = check_shape(M, K, group)) return rc;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    if (cfg && (cfg->flags & ~SPQT_CFG_Y_FP16)) return SPQT_EINVAL;
    const int y_half = cfg && (cfg->flags & SPQT_CFG_Y_FP16) ? 1 : 0;
    if ((uintptr_t)packed_dev % 128 != 0 || (uintptr_t)x_dev % 2 != 0 || (uintptr_t)y_dev % (y_half ? 2 : 4) != 0)
        return SPQT_EALIGN;
    spqt_launch_cfg c;
    if (cfg && (cfg->splits || cfg->waves)) {
        choose_cfg(M, K, batch, &c);
        if (cfg->splits) c.splits = cfg->splits;
        if (cfg->waves) c.waves = cfg->waves;
    } else {
        default_shape(M, K, batch, &c);
    }
    if (c.waves != 4 && !(c.waves == 8 && batch >= 3)) return SPQT_EINVAL;
    if (c.splits < 1 || c.splits > SPQT_MAX_SPLITS) return SPQT_EINVAL;
    const size_t need = needed_bytes(M, K, batch, c.splits, false);
    uint32_t *ws = nullptr;
    if (c.splits > 1) {
        if (!workspace_dev) return SPQT_EINVAL;
        if (workspace_bytes < need) return SPQT_ESIZE;
        if ((uintptr_t)workspace_dev % 256 != 0) return SPQT_EALIGN;
        ws = (uint32_t *)workspace_dev;
    }
    const int T = (int)tiles(M);
    const int grid = grid_blocks(T, c.splits);
    const int mf = kernel_rows(M, group, y_half) | (own_sets ? kOwnSetsBit : 0);
    hipError_t err = launch_fused_rows(c.waves, batch, grid, (hipStream_t)stream, (const uint8_t *)packed_dev, (const uint16_t *)x_dev,
                                       threshold, (float *)y_dev, ws, (int)K, c.splits, T, mf);
    return err == hipSuccess ? SPQT_OK : SPQT_EHIP;
}

extern "C" int spqt_gemv(const void *packed_dev, int64_t M, int64_t K, int group, const void *x_dev,
                         int batch, const int32_t *idx_dev, const int32_t *count_dev, float *y_dev,
                         void *workspace_dev, size_t workspace_bytes, void *stream) {
    return spqt_gemv_ex(packed_dev, M, K, group, x_dev, batch, idx_dev, count_dev, y_dev, workspace_dev,
                        workspace_bytes, stream, nullptr);
}
