// Internal helpers shared by the library's translation units (not part of the C ABI).
#ifndef SPQT_INTERNAL_H
#define SPQT_INTERNAL_H

#include <stdint.h>

#include "spqt.h"

namespace spqt {

constexpr int kTileRows = SPQT_TILE_ROWS;          // R: rows per zigzag tile
constexpr int kGroup = SPQT_GROUP;                 // G: columns per quantization group
constexpr int kScaleBytes = 2 * kTileRows;         // fp16 scales at the head of a chunk
constexpr int kColBytes = kTileRows / 2;           // one column of one tile: 128 bytes
constexpr int kChunkBytes = SPQT_CHUNK_BYTES;      // kScaleBytes + kGroup * kColBytes
static_assert(kChunkBytes == kScaleBytes + kGroup * kColBytes, "chunk size");

// Block-rows of a matrix with M rows; the last one is zero-padded when M is not a multiple of 256.
inline int64_t tiles(int64_t M) { return (M + kTileRows - 1) / kTileRows; }

// Bytes reserved at the head of the workspace: word 0 is the poison flag the reducers raise when a
// wait for partial sums is abandoned; the rest keeps the exchange words 256-byte aligned.
constexpr int kWorkspaceHead = 256;

// Bytes asked for where a launch with S workgroups per block-row brings just its exchange words (8 bytes for each of the
// `rows` outputs per block-row and activation row; the words are 32-bit, so half of it stays unused), head included.
inline size_t exchange_bytes(int64_t n_tiles, int rows, int S, int batch) {
    return kWorkspaceHead + (size_t)n_tiles * (size_t)rows * (size_t)S * (size_t)batch * 8;
}

// Bytes of one chunk (block-row t, group g) of the group layout: 256 fp16 scales + `group` column runs.
inline int chunk_bytes(int group) { return kScaleBytes + group * kColBytes; }

inline int check_shape(int64_t M, int64_t K, int group) {
    if (group != kGroup && group != kGroup / 2) return SPQT_ESHAPE;
    if (M <= 0 || K <= 0 || K % kGroup != 0) return SPQT_ESHAPE;
    if (M > (int64_t)1 << 24 || K > (int64_t)1 << 24) return SPQT_ESHAPE;
    return SPQT_OK;
}

// ceil(2^32 / n): what the kernels divide by n with (n >= 2; 0 for n = 1, which they do not use).
inline uint32_t inverse_of(int n) { return (uint32_t)((((uint64_t)1 << 32) + (uint32_t)n - 1) / (uint32_t)n); }

// Columns that the slices of the one-launch kernel of the group layout (gemv.hip) are whole multiples of; 31 heights and widths, both group
// sizes, to the column / units.  One or two rows: 1, so that slices are as even as can be (681 x 8960 at 20 % 6.2 / 7.1 us, 11008 x 4096
// at 20 % 8.0 / 8.7, two rows at 40 % 8.5 / 9.2; up to 70 % sparsity 2 % faster on average; few kept columns want units, as a pass ends with its
// last group: two rows at 95 % 4 % slower on average, 11008 x 4096 6.2 / 5.7).  Three or four rows: a unit.  Their passes hold ONE quantization group, so a slice
// that begins and ends inside a unit takes a pass more than its units do (4 rows at 40 %: groups of 64, 5120 x 5120 10.6 / 8.8, 5321 x 1920 8.6 / 7.4;
// groups of 128, 13678 x 2816 11.0 / 9.5, 11001 x 4224 11.4 / 10.0; 5 % faster on average, and 1 % slower where units make the longest slice half a pass
// longer, 13824 x 5120 12.9 / 13.0, 4096 x 14336 12.1 / 12.2).  Without compaction a pass IS a unit.
constexpr int slice_quantum(int batch, bool compact) { return compact && batch <= 2 ? 1 : 64; }

// Workgroups in the grid of a group-layout launch (block_of in gemv_common.hpp says which is which).
inline int grid_blocks(int64_t T, int S) { return 8 * (int)((T / 8) * S + ((T % 8) * S + 7) / 8); }

// Launch shape of the group layout with workgroups of 4 wavefronts, measured on MI355X over the benchmark's matrices at
// 50 % sparsity and dense.  default_shape below starts from it; a caller's own shape overrides it.
// One or two activation rows: about one workgroup per CU - at most 256 in total - and S any
// integer up to 16.  More workgroups only shorten every wavefront's slice, and the fixed cost per wavefront (dependent
// prologue loads, pipeline fill, exchange of partial sums) outweighs the extra parallelism: dense 13824 x 5120 with 4 / 8
// / 16 workgroups per block-row 9.7 / 11.0 / 12.3 us, index list at 50 % 28672 x 8192 with 2 / 4 / 6 15.5 / 17.0 / 17.0.
// Three or four rows: about 512 workgroups, S a power of two.
inline void choose_cfg(int64_t M, int64_t K, int batch, spqt_launch_cfg *out) {
    const int64_t T = tiles(M), NG = K / kGroup;
    const int waves = 4;
    int64_t S = 1;
    if (batch <= 2) {
        S = 256 / T;
        S = S < 1 ? 1 : (S > 16 ? 16 : S);
        while (S > 1 && S * waves > 4 * NG) --S;
    } else {
        while (S * 2 <= 16 && S * 2 * T <= 512) S *= 2;
        // keep at least a quarter of a quantization group per wavefront
        while (S > 1 && S * waves > 4 * NG) S /= 2;
    }
    out->splits = (int)S;
    out->waves = waves;
    out->flags = 0;
}

// Workgroups (of 4 wavefronts) per block-row of the column-block kernels, any integer up to 16; T block-rows.  What counts is
// how full the last round over the 256 CUs is: `depth` workgroups per CU leave T * S <= 256 * depth.  Power-of-two S
// left it at 62 to 87 % of the CUs for most heights.  The lines were drawn by sweeps of the kernels with two buffers of weights (4-bit 132
// VGPRs, 8-bit 110); the figures are of the present ones (100 and 77), us at 50 % sparsity or dense, and where a line no longer pays that is said:
//   - one workgroup per CU is where every kernel starts: 4-bit, T = 20, 5120 x 13824 S = 16 / 12 list 9.2 / 8.1, dense 12.3 / 10.3;
//   - lists of 1 or 2 rows go deeper for a 3 % fuller last round (8-bit, T = 86, 11008 x 4096 S = 2 / 5 / 8 8.7 / 8.1 / 8.5; the third workgroup no
//     longer pays there, and 4-bit, T = 54, 13824 x 5120 S = 4 / 8 / 14 is 8.1 / 8.6 / 8.2), the others only for a 20 % fuller one, since two
//     workgroups on a CU cost them more than that (4-bit dense 13824 x 5120 S = 4 / 8 10.0 / 10.7, 4 rows 19.9 / 21.5);
//     (with one row colblock4_list_splits and colblock8_list_splits below take back what no longer pays);
//   - a list slice of 112 to 256 columns (1 or 2 rows) is a pass and a bit: two workgroups per CU (no longer a gain: 8-bit 4096 x 4096
//     S = 8 / 16 5.5 / 5.7; 4-bit 9000 x 2944 with 105 columns S = 7 / 14 5.9 / 6.0);
//   - dense slices of at most one pass, if 3 workgroups per CU reach that without a less full round (no longer a gain: 4-bit 11008 x 4096
//     S = 5 / 16 8.1 / 8.7, 9000 x 2944 S = 7 / 14 6.8 / 6.8);
//   - one launch: slices of more than 5 units take a second workgroup per CU, S being the smallest with the same number of units in the longest
//     slice.  That evened out passes of one unit each; with full passes (kept_ring.hpp) and slices that are split to the column one per CU is as fast
//     or faster (S = one per CU / this rule: 4-bit 28672 x 8192 16.2 / 17.0, 14848 x 10240 12.3 / 13.0, 6400 x 16896 at 40 % 11.2 / 12.7, 8-bit 4096 x 11008
//     8.2 / 8.4).  With one per CU S is not lowered like that: every workgroup less makes the longest slice longer (4-bit 8704 x 7424 at 20 %
//     S = 6 / 7 10.1 / 9.7, K-quant 5120 x 13824 at 40 % S = 11 / 12 9.7 / 9.4); a workgroup goes only where no slice has more than 64 columns without it.
//     A third workgroup per CU has to leave a fuller round after the second one's lowering, too (14848 x 10240, 4-bit S = 8 / 10 13.0 / 14.3, 8-bit with
//     58 block-rows 11.2 / 12.2).  More than 128 block-rows with slices of at most 5 units exchange nothing (S = 1): a fuller round is worth
//     less than the exchange (22016 x 1024 8-bit S = 1 / 4 5.7 / 6.0, 44032 x 1280 4-bit S = 1 / 3 7.0 / 8.1, K-quant 7.4 / 8.1);
//   - several rows with slices from 1024 columns on: two workgroups per CU (4-bit, 4 rows, 28672 x 8192 S = 2 / 4 51 / 46.5).
// max_depth 1 (2-bit): a second workgroup per CU does not pay (list 28672 x 8192 S = 4 / 8 / 9 14.2 / 15.4 / 14.8, 14336 x 4096 S = 9 / 16 7.7 / 8.2;
// dense 24576 x 2048 S = 5 / 10 8.1 / 8.9, 14336 x 4096 S = 9 / 16 9.1 / 9.6, and where the last round is fuller 28672 x 8192 S = 4 / 9 20.3 / 19.7).
enum class Columns { list, dense, units };    // units: one launch, static ranges of columns
inline int colblock_splits(int64_t T, int64_t K, Columns from, int batch, int max_depth) {
    auto deepest = [&](int64_t depth) {
        const int64_t S = 256 * depth / T;
        return (int)(S < 1 ? 1 : (S > 16 ? 16 : S));
    };
    auto fill = [&](int64_t S) {              // per cent of the CUs' slots, rounds up to the last one
        const int64_t n = T * S, rounds = (n + 255) / 256;
        return (int)(n * 100 / (256 * rounds));
    };
    auto slice = [&](int64_t S) { return K / (4 * S); };
    const int64_t least_gain = from == Columns::list && batch <= 2 ? 103 : 120;
    int64_t S = deepest(1), depth = 1;
    const bool long_slices = from == Columns::units ? slice(S) > 5 * 64 : batch >= 2 && slice(S) >= 1024;
    if (from == Columns::units && T > 128 && !long_slices) return 1;
    if (max_depth >= 2 && long_slices) S = deepest(depth = 2);
    const int64_t units = K / 64;
    auto fewest = [&](int64_t s) {            // the smallest S with the same number of units in the longest slice
        while (s > 1 && (units + 4 * s - 1) / (4 * s) == (units + 4 * (s - 1) - 1) / (4 * (s - 1))) --s;
        return s;
    };
    for (int64_t d = depth + 1; d <= max_depth; ++d) {
        const int64_t gain = depth >= 2 ? 103 : least_gain;
        bool fuller = fill(deepest(d)) * 100 >= fill(S) * gain;
        if (from == Columns::units && depth >= 2) fuller = fuller && fill(fewest(deepest(d))) * 100 >= fill(fewest(S)) * gain;
        if (fuller) S = deepest(d);
    }
    if (max_depth >= 2 && from == Columns::list && batch <= 2 && slice(S) >= 112 && slice(S) <= 256 && T * S <= 256 && fill(deepest(2)) >= fill(S))
        S = deepest(2);
    if (from == Columns::dense && slice(S) > 64)
        for (int64_t d = 2; d <= max_depth; ++d)
            if (K <= 4 * 64 * deepest(d) && fill(deepest(d)) >= fill(S)) { S = deepest(d); break; }
    if (from != Columns::units) return (int)S;
    if (T * S > 256) return (int)fewest(S);
    while (S > 1 && 4 * 64 * (S - 1) >= K) --S;
    return (int)S;
}

// max_depth of the 4-bit layouts.  The K-quant kernel stages a minimum beside every scale: with 2 rows a CU held two of its workgroups while
// it had two buffers of weights (172 VGPRs), and the third that a list takes for a 3 % fuller round started a round of its own.  With one
// buffer (158 VGPRs, 42 KB of LDS) three fit, and the third loses or gains: 22016 x 1024 S = 5 / 8 7.4 / 8.4 us, 16896 x 4096 S = 7 / 11
// 12.3 / 12.6, but 13824 x 4096 S = 9 / 14 11.3 / 10.7, 14336 x 4096 S = 9 / 13 11.3 / 11.1.  Above 128 block-rows the split is so coarse that a finer one is worth
// it (35072 x 2048 S = 3 / 5 12.5 / 12.5, 43932 x 8192 S = 2 / 4 45 / 37).
inline int colblock4_depth(int64_t T, Columns from, int batch, bool kquant) {
    return kquant && from == Columns::list && batch == 2 && T <= 128 ? 2 : 3;
}

// max_depth of the 8-bit layout (figures of the present kernels; the lines were drawn with those of two buffers).  Dense, one row, 129 to 256
// block-rows, slices from 768 columns on: one workgroup per CU on two thirds of the CUs already reads at the rate of the memory, so a third
// workgroup per CU only adds the exchange (24576 x 8192 S = 1 / 4 35.9 / 37.2 us, 22016 x 4096 19.7 / 19.1, which was 18.2 / 19.1; below two thirds two per CU pay,
// 16640 x 8192 S = 1 / 3 35.0 / 28.3; short slices 22016 x 1024 S = 1 / 4 7.2 / 7.4).  One launch, more than 256 block-rows, fewer than 40 units: S = 1 / 2
// 33024 x 1536 9.3 / 9.3, 40960 x 1536 10.4 / 10.3, 36864 x 2304 13.4 / 13.0 (2816 columns 14.8 / 13.9 and 16.2 / 15.7; K-quant 66048 x 1536 11.9 / 11.3).
inline int colblock8_depth(int64_t T, int64_t K, Columns from, int batch) {
    if (from == Columns::units) return T > 256 && K < 2560 ? 2 : 3;
    return from == Columns::dense && batch == 1 && T > 128 && T <= 256 && K >= 4 * 768 ? 2 : 3;
}

// Workgroups per block-row of the 8-bit list kernel with one activation row, at most as many as `S`, what colblock_splits gives.  That rule was drawn with two
// buffers of weights; with one, a second and third workgroup per CU for a slightly fuller last round cost more in start and exchange than they
// bring.  Up to 128 block-rows: one per CU, two where they fill the last round a fifth better (S = this rule / before, us with the gather at 50 %:
// 9472 x 4096 S = 3 / 10 9.71 / 10.03, 9472 x 14336 18.8 / 19.6, 13440 x 8192 S = 2 / 7 16.3 / 16.9, 11008 x 4096 S = 5 / 8 10.2 / 10.6, 4096 x 8192 S = 8 / 16
// 9.48 / 9.74; slower by at most 1 %, 3072 x 4096 S = 10 / 16 7.72 / 7.66).  From 129 to 256 a block-row has one workgroup unless the idle CUs have much to
// read, K * (256 - T) above 400 thousand columns (S = 1 / 4: 23552 x 1152 7.6 / 8.2, 22016 x 4096, 344 thousand, 13.9 / 14.7, but 23552 x 8192, 590 thousand,
// 25.3 / 24.7; 17707 x 4096, 479 thousand, S = 1 / 5 13.2 / 12.9).  From 96 MB on the rule stays as it was: calls on one or two matrices of that size find
// kept columns in the 256 MB cache, where more requests in flight pay (13440 x 9728 at 70 %, S = 2 / 7, two matrices in turn 16.9 / 16.5, five 14.5 / 14.9).
inline int colblock8_list_splits(int64_t T, int64_t K, int S) {
    if (T > 256 || T * K >= (int64_t)96 * 8192) return S;         // (128 rows per block-row)
    if (T > 128) return K * (256 - T) <= 400000 ? 1 : S;
    const int64_t one = 256 / T, two = 512 / T;                   // one and two workgroups per CU
    const int64_t least = one * 6 * 2 <= two * 5 ? two : one;     // two * T of 512 slots against one * T of 256: fuller by a fifth
    return least < S ? (int)least : S;
}

// The same for the 4-bit list kernel with one activation row (not its K-quant flavour): up to 128 block-rows one workgroup per CU where that leaves slices of
// at most 256 columns.  Their sums are no further off than those of the shorter slices whatever is kept, since the first pass of a slice is centred and of four
// passes the second one too (gemv_cb.hip).  S = this rule / before, us with the gather and error against 64-bit arithmetic:
//   14336 x 4096   S = 4 / 9    at 50 %  9.44 / 9.96   1.63e-7 / 1.81e-7     all kept  11.7 / 12.8   2.00e-7 / 2.18e-7
//   11008 x 4096   S = 5 / 11   at 40 %  9.27 / 9.82   1.61e-7 / 1.80e-7     all kept  11.1 / 11.5   1.80e-7 / 2.08e-7
//   8192 x 8192    S = 8 / 16   at 50 %  10.1 / 10.9   1.71e-7 / 1.92e-7     all kept  12.8 / 13.3   2.07e-7 / 2.29e-7
// (no height slower by more than 0.5 %).  Longer slices would be 2 to 4 % faster and their sums further off (one pass centred, at 50 %: 14336 x 8192 12.4 / 12.8,
// 2.29e-7 / 2.10e-7; K-quant 14336 x 4096 9.58 / 9.87, 1.27e-7 / 1.24e-7).
inline int colblock4_list_splits(int64_t T, int64_t K, int S) {
    if (T > 128) return S;
    const int64_t one = 256 / T;
    return one < S && K <= 4 * 256 * one ? (int)one : S;
}

// A workspace the exchange can use: calls with several workgroups per block-row refuse any other.
inline bool usable_workspace(const void *ws, size_t bytes, size_t need) {
    return ws && bytes >= need && (uintptr_t)ws % 256 == 0;
}
// Whether a column-block call that asks for no launch shape and brings no usable workspace runs with ONE workgroup per
// block-row, which exchanges nothing.  Above these heights the block-rows alone keep the chip busy enough for that to be a
// sensible shape (half the CUs for a matrix of 64 MB and more and one row, all of them otherwise, twice that for a
// dense one, whose slices are shortest): 4-bit list at 50 % 33024 x 4096 without / with a workspace 14.5 / 12.0 us.
inline bool runs_without_workspace(int64_t T, size_t code_bytes, Columns from, int batch) {
    const bool large = batch == 1 && code_bytes >= (size_t)64 << 20;
    return T > (large ? 128 : (from == Columns::dense && batch == 1 ? 512 : 256));
}

// The launch shape of the group layout where the caller asks for none.
// Three or four activation rows, up to 256 block-rows: where choose_cfg's shape is more than one workgroup of 4 wavefronts per CU,
// the kernels run one workgroup of 8 per CU instead.  The exchange grows with rows times workgroups per block-row: index list at 70 %
// sparsity, 4 rows, 14336 x 4096 with 8 x 4 / 4 x 8 wavefronts per block-row 16.2 / 13.1 us, 28672 x 8192 with 4 x 4 / 2 x 8
// 30.3 / 26.7.  Higher matrices have nothing to exchange: 76800 x 1024 1 x 4 / 1 x 8 14.3 / 15.6, one launch 14.2 / 16.4.
inline void default_shape(int64_t M, int64_t K, int batch, spqt_launch_cfg *out) {
    const int64_t T = tiles(M);
    choose_cfg(M, K, batch, out);
    if (batch >= 3 && T <= 256 && T * out->splits > 256) {
        out->splits = (int)(256 / T);
        out->waves = 8;
    }
}

}  // namespace spqt
#endif
