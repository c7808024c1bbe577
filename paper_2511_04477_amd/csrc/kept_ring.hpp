// The one-launch mode of the column-block kernels (gemv_cb.hip, colblock_width.hpp), one activation row: where a wavefront's
// list entries come from when there is no list.
//
// Paper Section 2: a column is sparse iff |x_i| < threshold.  A wavefront's slice is a static range of columns (K split evenly,
// to the column).  It tests its range kRefillUnits units of 64 columns at a time, only as its passes need them, and compacts the
// kept columns into a ring of (column, x) entries in LDS: lane l tests the unit's column l, a ballot gives the kept set, mbcnt
// the rank.  A pass takes the next 64 entries of the ring as it takes 64 entries of an index list, so it is full whatever the
// sparsity; with one pass per unit, as it was, a pass had as many entries as its unit kept, and slices were whole units.
// Measured before / now (us, with the single buffer of weights in the kernels): 50 %, 4-bit 11008 x 4096 8.4 / 7.1, 4096 x 11008
// 8.0 / 7.4, 28672 x 8192 18.4 / 17.5; 8-bit 11008 x 4096 9.6 / 8.9; 2-bit 5120 x 13824 11.4 / 9.5; 40 %, K-quant 13824 x 5120 10.8 / 9.6,
// 5120 x 13824 11.3 / 9.7; 75 %, 8-bit 9088 x 12160 13.6 / 10.6.  Three units per refill: with two, a slice of 128 to 192 columns
// at 75 % takes two passes (K-quant 512 x 11264, two / three 6.1 / 5.2); four were 1 % slower than two over 60 shapes when the kernels had two buffers.
#ifndef SPQT_KEPT_RING_HPP
#define SPQT_KEPT_RING_HPP

#include "gemv_common.hpp"

namespace spqt {

constexpr int kRefillUnits = 3;
constexpr int kRingEntries = 512;         // a refill adds at most 192 to at most 63 live ones
constexpr int kRingSlots = kRingEntries + 64;   // dropped columns go behind the ring, which keeps the code free of branches

struct KeptRing {
    u32x2 *slots;                // LDS of this wavefront: {column, x bits}
    const uint16_t *x;
    int K, end;                  // columns of x, end of the slice
    float thr;
    int lane;
    int u;                       // first column not yet tested
    int filled = 0;              // entries written so far
    uint16_t xr[kRefillUnits] = {};

    __device__ __forceinline__ KeptRing(u32x2 *slots_, const uint16_t *x_, int K_, int begin, int end_, float thr_, int lane_)
        : slots(slots_), x(x_), K(K_), end(end_), thr(thr_), lane(lane_), u(begin) {}

    // Requests this lane's x of the units that the next refill tests (index clamped: values past the slice are unused).  Atomic
    // loads (the same instructions): the compiler moves plain ones behind the weights, to the use of their values.
    __device__ __forceinline__ void fetch() {
#pragma unroll
        for (int i = 0; i < kRefillUnits; ++i) {
            const int c = u + i * kPassCols + lane;
            xr[i] = __hip_atomic_load(x + (c < K ? c : K - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
    __device__ __forceinline__ void refill() {
#pragma unroll
        for (int i = 0; i < kRefillUnits; ++i) {
            const int c = u + i * kPassCols + lane;
            const bool keep = c < end && !(__builtin_fabsf(half_bits_to_float(xr[i])) < thr);
            const uint64_t mask = __ballot(keep);
            const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            slots[keep ? (filled + rank) & (kRingEntries - 1) : kRingEntries + lane] = u32x2{(uint32_t)c, (uint32_t)xr[i]};
            filled += (int)__popcll(mask);
        }
        filled = __builtin_amdgcn_readfirstlane(filled);
        u += kRefillUnits * kPassCols;
        __builtin_amdgcn_wave_barrier();
    }
    // Entry p + lane for the pass that starts at entry p (past the pass's n entries: anything).  One refill at most, so a pass
    // takes what is there (nothing, if kRefillUnits units keep nothing); the next x is requested every time, so that the number of
    // loads in flight is the same on every path.
    __device__ __forceinline__ u32x2 take(int p, int &n) {
        if (filled < p + kPassCols && u < end) refill();
        fetch();
        n = filled - p < kPassCols ? filled - p : kPassCols;
        return slots[(p + lane) & (kRingEntries - 1)];
    }
    __device__ __forceinline__ bool more(int p) const { return p < filled || u < end; }
};

}  // namespace spqt
#endif
