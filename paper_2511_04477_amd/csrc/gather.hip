// spqt_gather: threshold the hidden state and compact the surviving column indices.
//
// Paper Section 4.2.3 ("Sparse index collecting kernel design"): a binary mask of the
// entries that pass the threshold is prefix-summed and every active entry writes its index
// to the position the scan gives it, so the list is contiguous.  The paper scans 1024-entry
// segments with a Blelloch scan and orders the segments through a global atomic counter,
// which makes the order depend on arrival.  Here the list must be ascending and
// reproducible, so there are no atomics: workgroup b owns the 4096-entry segment b of x, 4 entries per lane, ranks its
// kept entries with wave64 primitives (ballot + mbcnt, the wavefronts' totals through LDS), and obtains its base offset by
// counting the kept entries of all earlier segments itself (x is at most 128 KB per row and sits in L2; counting is
// integer work on pairs of halves, the rows of a batch joined by a maximum before the test).
//
// What bounds it: the chain launch -> x -> ballot -> LDS -> list for one segment; for many, the last workgroup's read of
// all of x through one CU (64 bytes a clock).  Two entries per packed instruction and 16 wavefronts of 4 entries per
// lane, against fp32 compares and 8 wavefronts of 8 before: added time per call in a chain of GEMVs (an empty kernel adds
// 1.4 to 2.2 us) K = 4096 2.7 -> 2.4 us, 14336 3.7 -> 3.0, 28672 4.2 -> 3.6; 4 rows, 28672 10.0 -> 4.9.  (Requesting four
// chunks of the earlier segments at once instead of two: 14336 3.4, 28672 3.8.)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "keep.hpp"
#include "spqt_internal.h"

namespace {

using namespace spqt;

constexpr int kPerLane = 4;                        // own entries per lane: one 8-byte load of fp16 per row
constexpr int kMaxWaves = 16;
constexpr int kSegment = kMaxWaves * 64 * kPerLane;    // entries one workgroup ranks: 4096
constexpr int kCountCols = kMaxWaves * 64 * 8;         // entries of earlier segments a workgroup counts at a time: 8192

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// MASKED: besides the union list, write a copy of x in which every row has ITS OWN dropped
// entries set to zero.  A GEMV over the union list fed this copy gives each row the sum over
// that row's kept columns only (a dropped entry of a listed column contributes 0 * w).
// One workgroup of 1024 lanes per segment; a single segment may have fewer lanes (K <= 4 * lanes).
template <int BATCH, bool MASKED>
__global__ __launch_bounds__(kMaxWaves * 64) void spqt_gather_kernel(const uint16_t *__restrict__ x, int K, float thr,
                                                                     int32_t *__restrict__ idx, int32_t *__restrict__ count,
                                                                     uint16_t *__restrict__ x_masked) {
    __shared__ int wave_kept[kMaxWaves];
    __shared__ int wave_before[kMaxWaves];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int waves = blockDim.x >> 6;
    const int seg = blockIdx.x;
    const int first = seg * kSegment + (int)threadIdx.x * kPerLane;
    const bool inside = first < K;                 // K % 8 == 0: a lane's entries are all inside x or all past its end

    u32x2 v[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) v[b] = *reinterpret_cast<const u32x2 *>(x + (size_t)b * K + (inside ? first : 0));

    // Kept entries of all earlier segments, counted by this workgroup itself.
    const uint32_t c2 = threshold_bits(thr);
    int before = 0;
    const int upto = seg * kSegment;
#pragma unroll 2
    for (int p = (int)threadIdx.x * 8; p < upto; p += kCountCols) {
        u32x4 m = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const u32x4 e = *reinterpret_cast<const u32x4 *>(x + (size_t)b * K + p);
#pragma unroll
            for (int d = 0; d < 4; ++d) m[d] = b == 0 ? magnitude_bits(e[d]) : larger_bits(m[d], magnitude_bits(e[d]));
        }
        before += 8 - (int)__popc(dropped_signs(m.x, c2) | (dropped_signs(m.y, c2) >> 1) | (dropped_signs(m.z, c2) >> 2) |
                                  (dropped_signs(m.w, c2) >> 3));
    }

    uint32_t m0 = 0u, m1 = 0u;
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        const uint32_t a0 = magnitude_bits(v[b].x), a1 = magnitude_bits(v[b].y);
        m0 = b == 0 ? a0 : larger_bits(m0, a0);
        m1 = b == 0 ? a1 : larger_bits(m1, a1);
        if (MASKED && inside) {
            // a dropped half's sign bit, brought down to bit 0 of its half, times 0xFFFF covers the half
            const uint32_t t0 = dropped_signs(a0, c2) >> 15, t1 = dropped_signs(a1, c2) >> 15;
            *reinterpret_cast<u32x2 *>(x_masked + (size_t)b * K + first) = u32x2{v[b].x & ~((t0 << 16) - t0), v[b].y & ~((t1 << 16) - t1)};
        }
    }
    const uint32_t d0 = dropped_signs(m0, c2), d1 = dropped_signs(m1, c2);
    const bool kept[kPerLane] = {inside && !(d0 & 0x8000u), inside && !(d0 >> 31), inside && !(d1 & 0x8000u), inside && !(d1 >> 31)};
    int rank = 0, total = 0;     // entries kept by lower lanes, and by the whole wavefront
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        const uint64_t ballot = __ballot(kept[j]);
        rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, (uint32_t)rank));
        total += __popcll(ballot);
    }
    if (seg > 0) before = wave_total(before);
    if (lane == 0) {
        wave_kept[wave] = total;
        wave_before[wave] = before;
    }
    __syncthreads();
    const int w = lane < waves ? lane : 0;
    const int wk = lane < waves ? wave_kept[w] : 0, wb = lane < waves ? wave_before[w] : 0;
    const int base = wave_total(wb + (lane < wave ? wk : 0));
    if (seg == (int)gridDim.x - 1 && wave == waves - 1 && lane == 0) *count = base + total;

    int pos = base + rank;
#pragma unroll
    for (int j = 0; j < kPerLane; ++j)
        if (kept[j]) idx[pos++] = first + j;
}

int run_gather(const void *x_dev, int64_t K, int batch, float threshold, int32_t *idx_out_dev,
               int32_t *count_out_dev, void *x_masked_dev, void *stream) {
    if (!x_dev || !idx_out_dev || !count_out_dev) return SPQT_EINVAL;
    if (K <= 0 || K % kGroup != 0 || K > SPQT_GATHER_MAX_K) return SPQT_ESHAPE;
    if (batch < 1 || batch > SPQT_MAX_BATCH) return SPQT_ESHAPE;
    if (threshold != threshold) return SPQT_EINVAL;   // NaN threshold has no meaning
    if ((uintptr_t)x_dev % 16 != 0 || (uintptr_t)idx_out_dev % 4 != 0) return SPQT_EALIGN;
    if ((uintptr_t)x_masked_dev % 16 != 0) return SPQT_EALIGN;
    const int segments = (int)((K + kSegment - 1) / kSegment);
    const dim3 grid(segments), block(segments > 1 ? kMaxWaves * 64 : 64 * (int)((K + 64 * kPerLane - 1) / (64 * kPerLane)));
    hipStream_t st = (hipStream_t)stream;
    const uint16_t *x = (const uint16_t *)x_dev;
    if (x_masked_dev) {
        uint16_t *xm = (uint16_t *)x_masked_dev;
        switch (batch) {
            case 1: hipLaunchKernelGGL((spqt_gather_kernel<1, true>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, xm); break;
            case 2: hipLaunchKernelGGL((spqt_gather_kernel<2, true>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, xm); break;
            case 3: hipLaunchKernelGGL((spqt_gather_kernel<3, true>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, xm); break;
            default: hipLaunchKernelGGL((spqt_gather_kernel<4, true>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, xm); break;
        }
        return hipGetLastError() == hipSuccess ? SPQT_OK : SPQT_EHIP;
    }
    switch (batch) {
        case 1: hipLaunchKernelGGL((spqt_gather_kernel<1, false>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, (uint16_t *)nullptr); break;
        case 2: hipLaunchKernelGGL((spqt_gather_kernel<2, false>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, (uint16_t *)nullptr); break;
        case 3: hipLaunchKernelGGL((spqt_gather_kernel<3, false>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, (uint16_t *)nullptr); break;
        default: hipLaunchKernelGGL((spqt_gather_kernel<4, false>), grid, block, 0, st, x, (int)K, threshold, idx_out_dev, count_out_dev, (uint16_t *)nullptr); break;
    }
    return hipGetLastError() == hipSuccess ? SPQT_OK : SPQT_EHIP;
}

}  // namespace

extern "C" int spqt_gather(const void *x_dev, int64_t K, int batch, float threshold,
                           int32_t *idx_out_dev, int32_t *count_out_dev, void *stream) {
    return run_gather(x_dev, K, batch, threshold, idx_out_dev, count_out_dev, nullptr, stream);
}

extern "C" int spqt_gather_rows(const void *x_dev, int64_t K, int batch, float threshold,
                                int32_t *idx_out_dev, int32_t *count_out_dev, void *x_masked_out_dev,
                                void *stream) {
    if (!x_masked_out_dev || !x_dev) return SPQT_EINVAL;
    if (K > 0 && batch > 0) {   // the copy may not overlap x: other workgroups are still reading it
        const uintptr_t a = (uintptr_t)x_dev, b = (uintptr_t)x_masked_out_dev;
        const uintptr_t bytes = (uintptr_t)K * (uintptr_t)batch * 2u;
        if (a < b + bytes && b < a + bytes) return SPQT_EINVAL;
    }
    return run_gather(x_dev, K, batch, threshold, idx_out_dev, count_out_dev, x_masked_out_dev, stream);
}
