// The sparsity test on fp16 bit patterns, shared by the gather kernel and the one-launch kernel with even shares.
#ifndef SPQT_KEEP_HPP
#define SPQT_KEEP_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spqt {

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// For an fp16 x and an fp32 thr, |x| < thr holds iff |x| < c, c being the smallest fp16 value >= thr (c = 0 for thr <= 0:
// nothing is below it; c = +inf for thr above the largest finite fp16), and for non-negative fp16 values the order of the
// values is the order of their bit patterns, NaN patterns lying above +inf: so the test is (bits & 0x7FFF) < bits(c)
// as 15-bit integers, two halves of a dword at a time - exactly the result of the fp32 comparison
// (NaN and, at any finite threshold, Inf are kept; an entry equal to the threshold is kept).
// Returns bits(c) in both halves.
__device__ __forceinline__ uint32_t threshold_bits(float thr) {
    if (!(thr > 0.0f)) return 0u;
    const _Float16 h = (_Float16)thr;                       // round to nearest even
    uint32_t b = __builtin_bit_cast(uint16_t, h);
    if ((float)h < thr) b += 1u;                            // next fp16 up (from the largest finite one: +inf)
    return b | (b << 16);
}
__device__ __forceinline__ uint32_t magnitude_bits(uint32_t two_halves) { return two_halves & 0x7FFF7FFFu; }
// The larger magnitude of each half: a column of several rows is kept iff its largest magnitude passes the test.
__device__ __forceinline__ uint32_t larger_bits(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
// Sign bits (bit 15 / bit 31) set where the half with this magnitude is DROPPED.
__device__ __forceinline__ uint32_t dropped_signs(uint32_t magnitudes, uint32_t c2) {
    const s16x2 d = __builtin_bit_cast(s16x2, magnitudes) - __builtin_bit_cast(s16x2, c2);
    return __builtin_bit_cast(uint32_t, d) & 0x80008000u;
}

// Sum over the 64 lanes (wave-uniform).
__device__ __forceinline__ int wave_total(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    return __builtin_amdgcn_readlane(v, 15) + __builtin_amdgcn_readlane(v, 31) + __builtin_amdgcn_readlane(v, 47) +
           __builtin_amdgcn_readlane(v, 63);
}

}  // namespace spqt
#endif
