// How a launch divides its work: which workgroup of which block-row a launch index is, and which part of the columns a wavefront
// takes.  Integer arithmetic alone, for the device and, where a test compiles it, the host.
#ifndef SPQT_SPLIT_HPP
#define SPQT_SPLIT_HPP

#include "spqt_internal.h"

#ifdef __HIPCC__
#define SPQT_BOTH __host__ __device__ __forceinline__
#else
#define SPQT_BOTH inline
#endif

namespace spqt {

SPQT_BOTH uint32_t mul_hi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }

// Which workgroup of which block-row a launch index is.  Workgroups go to the 8 XCDs round-robin by index; the S workgroups
// of a block-row are kept on ONE XCD as far as that leaves the XCDs equally loaded: block-rows in multiples of 8 go to the
// XCDs whole, and the workgroups of the T % 8 that are left are spread over the XCDs evenly (with 20 block-rows, whole
// ones would give four XCDs 3 and four 2: 5120 x 13824 dense, 12 workgroups per block-row, 13.1 us, evenly 10.4).  A
// spread block-row's reducer may run before producers on another XCD are dispatched, which combine_block_row allows for.
// Returns false for the padding of the grid (grid_blocks).
SPQT_BOTH bool is_spread(int t, int T) { return t >= (T & ~7); }
// inv: inverse_of(S * WAVES).
template <int WAVES>
SPQT_BOTH bool block_of(uint32_t index, int S, int T, uint32_t inv, int &t, int &s) {
    const uint32_t xcd = index & 7u;
    const uint32_t slot = index >> 3;                                          // position among this XCD's workgroups
    const uint32_t whole = ((uint32_t)T >> 3) * (uint32_t)S;                   // workgroups of whole block-rows per XCD
    const uint32_t left = ((uint32_t)T & 7u) * (uint32_t)S;
    const uint32_t per_xcd = (left + 7u) >> 3;
    const bool in_whole = slot < whole;
    const uint32_t r = in_whole ? slot : xcd * per_xcd + slot - whole;         // one division serves both
    // r / S; the rounded-up inverse gives it exactly while r * WAVES * (S * WAVES) < 2^32.  M <= 2^24 and S <= 64: r < 2^20 with block-rows
    // of 128 rows (at most 4 wavefronts), r < 2^19 with higher ones (at most 8)
    const uint32_t q = WAVES == 1 ? r / (uint32_t)S : mul_hi(r * (uint32_t)WAVES, inv);
    t = (int)(in_whole ? xcd + 8u * q : ((uint32_t)T & ~7u) + q);
    s = (int)(r - q * (uint32_t)S);
    return in_whole || (slot - whole < per_xcd && r < left);
}

// Part `part` of `parts` equal parts of n things: [floor(n * part / parts), floor(n * (part + 1) / parts)).  In 32-bit
// arithmetic for every n <= 2^24 and parts <= 512: with n = q * parts + r a part starts at q * part + floor(r * part / parts).
// The divisions are products with inv = inverse_of(parts), rounded up: exact for r * part < 2^18, and for n the quotient may be
// one too large (with more than 256 parts and n > 2^23), which shows as a negative remainder.
struct Share {
    int begin, end;
};
template <int WAVES>
SPQT_BOTH Share share_of(int n, int part, int parts, uint32_t inv) {
    int q, r;
    if (WAVES == 1) {              // parts may be 1, which has no 32-bit inverse
        q = (int)((uint32_t)n / (uint32_t)parts);
        r = n - q * parts;
        return {q * part + (int)((uint32_t)(r * part) / (uint32_t)parts), q * (part + 1) + (int)((uint32_t)(r * (part + 1)) / (uint32_t)parts)};
    }
    q = (int)mul_hi((uint32_t)n, inv);
    r = n - q * parts;
    q -= r < 0 ? 1 : 0;
    r += r < 0 ? parts : 0;
    return {q * part + (int)mul_hi((uint32_t)(r * part), inv), q * (part + 1) + (int)mul_hi((uint32_t)(r * (part + 1)), inv)};
}

}  // namespace spqt
#endif
