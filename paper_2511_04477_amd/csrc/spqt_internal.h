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
inline size_t counter_bytes(int64_t) { return 256; }

// Bytes of exchange words a launch with S workgroups per block-row really touches (64-bit words,
// `rows` outputs per block-row and activation row), head included.
inline size_t exchange_bytes(int64_t n_tiles, int rows, int S, int batch) {
    return 256 + (size_t)n_tiles * (size_t)rows * (size_t)S * (size_t)batch * 8;
}

// Bytes of one chunk (block-row t, group g) of the group layout: 256 fp16 scales + `group` column runs.
inline int chunk_bytes(int group) { return kScaleBytes + group * kColBytes; }

inline int check_shape(int64_t M, int64_t K, int group) {
    if (group != kGroup && group != kGroup / 2) return SPQT_ESHAPE;
    if (M <= 0 || K <= 0 || K % kGroup != 0) return SPQT_ESHAPE;
    if (M > (int64_t)1 << 24 || K > (int64_t)1 << 24) return SPQT_ESHAPE;
    return SPQT_OK;
}

// Workgroups in the grid of a group-layout launch (block_of in gemv_common.hpp says which is which).
inline int grid_blocks(int64_t T, int S) { return 8 * (int)((T / 8) * S + ((T % 8) * S + 7) / 8); }

enum class Kernel { group_layout, colblock_list, colblock_dense };

// Launch shape, measured on MI355X over the benchmark's matrices at 50 % sparsity and dense.
// Group layout, one or two activation rows: about one workgroup of 4 wavefronts per CU - at most 256 in total - and S any
// integer up to 16.  More workgroups only shorten every wavefront's slice, and the fixed cost per wavefront (dependent
// prologue loads, pipeline fill, exchange of partial sums) outweighs the extra parallelism: dense 13824 x 5120 with 4 / 8
// / 16 workgroups per block-row 9.7 / 11.0 / 12.3 us, index list at 50 % 28672 x 8192 with 2 / 4 / 6 15.5 / 17.0 / 17.0.
// Three or four rows, and the column-block layouts: about 512 (dense with one row: 1024) workgroups, S a power of two.
inline void choose_cfg(int64_t M, int64_t K, int batch, Kernel kind, spqt_launch_cfg *out) {
    const int64_t T = tiles(M), NG = K / kGroup;
    const int waves = 4;
    int64_t S = 1;
    if (kind == Kernel::group_layout && batch <= 2) {
        S = 256 / T;
        S = S < 1 ? 1 : (S > 16 ? 16 : S);
        while (S > 1 && S * waves > 4 * NG) --S;
    } else {
        const bool big = (size_t)M * (size_t)K / 2 >= ((size_t)64 << 20);
        const int64_t target = batch >= 2 ? 512 : (kind != Kernel::colblock_dense ? 512 : (big ? 256 : 1024));
        while (S * 2 <= 16 && S * 2 * T <= target) S *= 2;
        // keep at least a quarter of a quantization group per wavefront
        while (S > 1 && S * waves > 4 * NG) S /= 2;
    }
    out->splits = (int)S;
    out->waves = waves;
    out->flags = 0;
}

// Three or four activation rows: where choose_cfg's shape is more than one workgroup of 4 wavefronts per CU, the kernels run
// one workgroup of 8 per CU instead.  The exchange grows with rows times workgroups per block-row: index list at 70 %
// sparsity, 4 rows, 14336 x 4096 with 8 x 4 / 4 x 8 wavefronts per block-row 16.2 / 13.1 us, 28672 x 8192 with 4 x 4 / 2 x 8
// 30.3 / 26.7.  (spqt_default_cfg and the limit of spqt_gemv_static go by choose_cfg's shape, which never needs fewer
// exchange words.)
inline void wide_workgroups(int64_t M, int batch, spqt_launch_cfg *c) {
    const int64_t T = tiles(M);
    if (batch < 3 || T * c->splits <= 256) return;
    c->splits = T < 256 ? (int)(256 / T) : 1;
    c->waves = 8;
}

}  // namespace spqt
#endif
