// One pass of the group-layout GEMV kernels: up to 64 columns of a block-row, 128 bytes each, multiplied on the
// matrix cores for 1..4 activation rows.  Shared by gemv_list.hip (index list, dense), gemv.hip (one launch, static
// column ranges) and gemv_bal.hip (one launch, even shares).
//
// Slots: entry e of a pass sits in slot (c, u), c = e / 4 % 4, u = e / 16 * 4 + e % 4, so that 16 entries are four slots of every quarter and
// a pass of few entries leaves out the products of the sixteens it does not reach.  In step u the
// 16 lanes of quarter c of the wavefront read the 128-byte run of column (c, u), 8 bytes each: lane l holds rows
// 16 n .. 16 n + 15 of the block-row, n = l % 16, at the 16 columns of its quarter.  Lane e deals entry e; its column's offset
// moves to lane (c, u) once (slot_order), i.e. into the quarter that reads it, and from there to the other 15 lanes by DPP
// (row_newbcast).
// What bounds a pass: its instructions, where a SIMD holds one wavefront (2 ns each).  About 500 of them became 420 when the masked A came to be read
// from LDS, the sign of x to be undone by the addend of the next pass, and scales to be found with one v_readlane each (index list at 50 %
// 28672 x 8192 16.4 / 15.8 us, one launch at 40 % 11008 x 4096 7.28 / 7.07), and 400 when the two rows that share a dword came to be told apart by A, not by
// pairing the halves of two columns (before / now, us: dense 5120 x 5120 6.37 / 6.16, 13824 x 5120 8.97 / 8.67, 5120 x 13824 9.30 / 8.98; with a list or in one
// launch, whose slices also wait for entries, 0 to 1 %: 4096 x 14336 at 50 % with the gather 9.48 / 9.40; 4 rows 28672 x 8192 at 70 % 26.8 / 26.65).
// Two passes' weights requested ahead of the products (a second buffer) were 3 to 6 % slower: the memory, not the order of the requests, sets
// when the second pass arrives.
// Slices end with a short pass: leaving half of its products out took chains of GEMVs from 356.7 to 353.1 us (one launch, 48 of 11008 x 4096 and its
// transpose, 40 %), 208.6 to 205.0 (two rows with their own sets, 24 of 14336 x 4096 and its transpose) and 166.9 to 164.9 (four rows, 6 of
// 28672 x 8192 and its transpose).  By sixteens instead of halves, before / now: list with the gather 4096 x 4096 at 50 % (32 or 33 entries per
// wavefront) 7.13 / 7.04, at 40 % 7.53 / 7.40, 4 rows at 70 % 8192 x 28672 27.0 / 26.8, one launch at 40 % 11008 x 4096 6.88 / 6.81.
//
// Products: v_mfma_f32_16x16x32_f16 computes D[m][n] += sum over 32 k of A[m][k] * B[k][n]; lane l brings A[l % 16] and
// B[..][l % 16] at the 8 k of quarter l / 16, i.e. at 4 of the 16 columns of its quarter with two k each, h = 0 and 1.  B is one dword of each
// column, shifted and masked: the halves are ONE code each, of two rows of W.  A is the raw fp16 x, in row m at the k of the half
// that row m is about and zero at the other: the two rows that share a dword need not be brought apart.
// The sum over k is the sum over all columns of the pass, so nothing is left to fold across lanes.
// The 16 rows of A are 4 v + j: v = 2 d + h (d: which dword of the column, two variants of A with zeros in the other rows; h: which half) says which
// four of the lane's 16 rows of W the product belongs to, so that all 16 rows end up in FOUR accumulator tuples D[p], and j = 0..3 separates
// activation rows and quantization groups (j = group of the pass * rows + activation row): one activation row takes
// columns of up to 4 groups per pass, two rows 2 groups, three or four rows one.  Lane (v, n) = (l / 16, l % 16) ends
// up with rows 16 n + 4 v + p, p = 0..3, in D[p][j]; the group's scale is applied there and the lane's 4 outputs per
// activation row are all that is carried from pass to pass.
//
// Why this form: with 4-wide products (v_mfma_f32_4x4x4) a lane keeps 32 sums per activation row that must be folded
// over 8 lanes - per pass, when a pass is one group, or once per slice at the price of 32 scales per lane and pass.
// That took 244 VGPRs for 4 rows and 218 for one (two wavefronts per SIMD) and made the kernels issue-bound.  Measured before
// and after (us, HIP graph, weights cold): index list at 50 %, one row 14336 x 4096 9.0 / 7.8, 28672 x 8192 16.6 / 15.6; 4 rows
// at 70 % 14336 x 4096 18.3 / 13.5, 28672 x 8192 32.9 / 27.0; one launch, 2 rows at 65 %, 28672 x 8192 25.1 / 20.0; dense
// 5120 x 13824 13.3 / 10.0 (half of that from the launch shape).  What bounds them now: the fixed cost of a launch (start,
// first weights, exchange: about 5 us) on small matrices, HBM on large ones (28672 x 8192 dense: 5.3 TB/s).
#ifndef SPQT_PASS_HPP
#define SPQT_PASS_HPP

#include "gemv_common.hpp"

namespace spqt {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f16x8 as_f16x8(u32x4 bits) { return __builtin_bit_cast(f16x8, bits); }

// Where the four codes of 16 bits of a column run are multiplied, and what undoes the units: codes 1 and 3 at bits 7..10 of an fp16 half (code * 2^-17;
// from code 8 on the half has exponent field 1, whose step is the subnormals' 2^-24 too), codes 0 and 2 at bits 3..6 (code * 2^-21).  Codes 0 and 1 are
// shifted left by 3, codes 2 and 3 right by 5.
constexpr float kUnit[4] = {2097152.0f, 131072.0f, 2097152.0f, 131072.0f};

// activation rows as the passes count them (3 is treated as 4 with a zero row), and quantization groups per pass
constexpr int padded_rows(int batch) { return batch == 3 ? 4 : batch; }
constexpr int groups_per_pass(int batch) { return 4 / padded_rows(batch); }

// x of the 64 slots of a pass as fp16, a dword per slot: rows 2 j + h, j as above, x in the lower (h = 0) or the upper half (h = 1) of the
// dword and zero in the other; rows 8 and 9 take what no product reads.  A row is 16 bytes longer than its slots, so that the 8 rows that are
// read together lie in different banks.
struct StagedX {
    uint32_t v[10][kPassCols + 4];
    uint32_t zeros[16];
};
// Where in StagedX a lane reads its part of A: the x of its row m = 8 d + 4 h + j at the 16 slots of its quarter, in the variant of A that is the
// lane's; zeros in the other.  (Reading the zeros costs one instruction per 16 bytes; masking what is read, four.)
struct ReadsX {
    const u32x4 *mine, *of_variant[2];
    __device__ __forceinline__ ReadsX(StagedX &xs, int lane) {
        if (lane < 16) xs.zeros[lane] = 0u;
        mine = reinterpret_cast<const u32x4 *>(&xs.v[2 * (lane & 3) + ((lane >> 2) & 1)][lane & 48]);
#pragma unroll
        for (int d = 0; d < 2; ++d) of_variant[d] = ((lane >> 3) & 1) == d ? mine : reinterpret_cast<const u32x4 *>(xs.zeros);
    }
};

// v of lane U of the caller's row of 16 lanes, in every lane of the row.
template <int U>
__device__ __forceinline__ uint32_t row_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + U, 0xf, 0xf, true);
}

// The slot (16 c + u) of the entry that lane e deals, and what a lane's slot gets: `v` of the lane that deals the slot's entry (the same
// permutation, which is its own inverse).
__device__ __forceinline__ int slot_of(int e) { return ((e & 0x0C) << 2) | ((e & 0x30) >> 2) | (e & 3); }
__device__ __forceinline__ uint32_t slot_order(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * slot_of(lane), (int)v); }

// Requests the weights of slots u = FROM .. TO - 1 of a pass: off = byte offset (from base) of the column run of the entry
// this lane owns, n8 = 8 * (lane % 16).
template <int FROM, int TO>
__device__ __forceinline__ void load_columns(const uint8_t *base, uint32_t off, uint32_t n8, u32x2 (&w)[16]) {
    w[FROM] = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(base + (size_t)(row_lane<FROM>(off) + n8)));
    if constexpr (FROM + 1 < TO) load_columns<FROM + 1, TO>(base, off, n8, w);
}

// Products of the 16 slots (c, u), u = 4 Q .. 4 Q + 3: d[p][j] += sum of code(row 16 n + 4 v + p, slot) * x(j, slot)
// in units of kUnit[p].
// The matrix cores align products by the exponent FIELDS, so bits that a half has above its code are bits of precision lost in every product: codes sit as
// high as one shift per two codes brings them.  That is by row, not only on the whole: error against 64-bit arithmetic of rows 0, 1, 2, 3 modulo 4,
// dense 5120 x 5120, 1.7e-7 9.4e-8 1.7e-7 9.2e-8 with Laplace x, 5.5e-7 1.0e-7 5.4e-7 1.0e-7 with SiLU products.  (Other places for six instructions: at bits 6, 4, 2,
// 6 with the bias at 2 2.6e-7 2.8e-7 5.4e-7 2.6e-7 - on 1024 x 5120 rows 0 were closer so, 1.3e-7, now 1.7e-7 -, at 7, 4, 3, 7 with SiLU products 1.1e-7 2.0e-7 5.4e-7 1.0e-7.  For seven, 7, 7, 3, 7, 1.1e-7 1.0e-7
// 5.4e-7 1.0e-7 and 0.5 to 1 % longer calls; for eight, all at bit 7, 1.0e-7 in every row and 1 to 3 %.)
template <int Q>
__device__ __forceinline__ void quarter_pass(const u32x2 (&w)[16], const ReadsX &rx, f32x4 (&d)[4]) {
    const u32x4 x[2] = {rx.of_variant[0][Q], rx.of_variant[1][Q]};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        u32x4 b[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t c = w[4 * Q + k][i], left = c << 3, right = c >> 5;
            b[0][k] = left & 0x00780078u;
            b[1][k] = left & 0x07800780u;
            b[2][k] = right & 0x00780078u;
            b[3][k] = right & 0x07800780u;
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) d[p] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(x[i]), as_f16x8(b[p]), d[p], 0, 0, 0);
    }
}

// The bias of the offset-binary codes (stored = q + 8) enters as the accumulators' initial value: the product of x with
// the constant -8 in the units of codes 1 and 3, where no bit of it is lost.
__device__ __forceinline__ void start_products(const ReadsX &rx, f32x4 (&d)[4]) {
    const f16x8 eight = as_f16x8(u32x4{0x84008400u, 0x84008400u, 0x84008400u, 0x84008400u});    // -8 * 2^-17
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(rx.mine[i]), eight, sum, 0, 0, 0);
    d[1] = d[3] = sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) d[0][j] = d[2][j] = sum[j] * (kUnit[1] / kUnit[0]);
}

// Every other pass is computed with -x.  The matrix cores round the terms of a product DOWN, so a
// sum over many passes carries a negative bias, relative to the result in proportion to sqrt(K).  With x negated the bias
// changes sign, so every other pass is negated and it cancels: against 64-bit arithmetic (relative 2-norm, 1024 x 28672
// dense, one row) 4.4e-6 -> 4.6e-7 for Laplace x and 1.3e-5 -> 7.8e-7 for SiLU products.  (The 4-wide products of
// v_mfma_f32_4x4x4 have a bias of the same sign, 1.1e-5 and 2.7e-5.)  The wavefronts of a block-row start with different signs,
// so slices of one pass cancel too.
constexpr uint32_t kSignOfX = 0x8000u;

// Applies the scales of a pass's groups (sc[g] = the fp16 scales of the lane's 4 rows in group g of the pass) and adds to
// the lane's running sums, which stay in the products' units.  The sums carry the sign of the pass's x: each pass subtracts the sums
// of those before it.
template <int BATCH, int GROUPS>
__device__ __forceinline__ void add_scaled(const f32x4 (&d)[4], const u32x2 (&sc)[GROUPS], float (&acc)[BATCH][4]) {
    constexpr int kRows = padded_rows(BATCH);
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const f16x2 h01 = as_f16x2(sc[g].x), h23 = as_f16x2(sc[g].y);
        const float s[4] = {(float)h01.x, (float)h01.y, (float)h23.x, (float)h23.y};
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
#pragma unroll
            for (int p = 0; p < 4; ++p) acc[b][p] = __builtin_fmaf(s[p], d[p][g * kRows + b], g == 0 ? -acc[b][p] : acc[b][p]);
    }
}

// The entries of a pass, dealt to its groups: lane e holds candidate column kk (or -1 past the slice), candidates are
// consecutive list entries, and a run of entries of one quantization group is one group of the pass.  A run that would
// be group GROUPS (counted from 0) waits for the next pass.
struct Deal {
    bool take;      // this lane's candidate belongs to the pass
    int j;          // its group inside the pass
    int n;          // entries the pass takes (wave-uniform): the next pass starts n entries further
    uint64_t starts;   // lanes at which the pass's groups start (wave-uniform)
};
template <int GROUPS>
__device__ __forceinline__ Deal deal_groups(int kk, int g, int lane) {
    Deal d;
    const bool cand = kk >= 0;
    const int gprev = __builtin_amdgcn_update_dpp(-1, g, 0x138, 0xf, 0xf, false);   // wave_shr:1; lane 0 keeps -1
    const uint64_t cands = __builtin_amdgcn_ballot_w64(cand);
    d.starts = __builtin_amdgcn_ballot_w64(g != gprev) & cands;
    if constexpr (GROUPS == 1) {                 // the pass ends where a second group starts (counting groups: 4 rows 8192 x 28672 at 70 % 28.5 / 28.3 us)
        const uint64_t second = d.starts & ~1ull;
        d.j = 0;
        d.n = second ? (int)__builtin_ctzll(second) : (int)__popcll(cands);
        d.take = lane < d.n;
        return d;
    }
    const uint64_t further = d.starts >> 1;      // counted below lane l: the starts at lanes 1 .. l
    d.j = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(further >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)further, 0u));
    d.n = (int)__popcll(__builtin_amdgcn_ballot_w64(d.j < GROUPS) & cands);
    d.take = lane < d.n;                         // candidates and groups come in the order of the lanes
    return d;
}

// Stages the x of a pass: the entry that lane `lane` deals, in its slot, carries x[b] for group j of the pass (4: none).
// Slots that no entry writes must read as zero: with one group per pass every lane writes its slot, and the rest is cleared once.
__device__ __forceinline__ void clear_x(StagedX &xs, int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) reinterpret_cast<u32x4 *>(xs.v[4 * i + (lane >> 4)])[lane & 15] = u32x4{0u, 0u, 0u, 0u};
    __builtin_amdgcn_wave_barrier();
}
template <int BATCH, int GROUPS>
__device__ __forceinline__ void stage_x(StagedX &xs, int lane, int j, uint32_t sign, const uint16_t (&xraw)[BATCH]) {
    constexpr int kRows = padded_rows(BATCH);
    if (GROUPS > 1) clear_x(xs, lane);
    // no branch on j: a divergent one inside the pipeline's loop makes the compiler join the loop's exits with its
    // entry and wait for all loads there
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        const uint16_t v = (uint16_t)(GROUPS > 1 || j < 4 ? xraw[b] ^ sign : 0u);
        // (with two rows and two groups the rows of group 4 would lie behind the array)
        const int row = GROUPS == 1 ? b : (kRows == 1 || j < 4 ? j * kRows + b : 4);
        uint16_t *at = reinterpret_cast<uint16_t *>(&xs.v[2 * row][slot_of(lane)]);
        at[0] = v;
        at[2 * (kPassCols + 4) + 1] = v;
    }
    __builtin_amdgcn_wave_barrier();
}

// What the HEAD of a pass leaves for its loads and its products.
template <int BATCH>
struct PassHead {
    uint32_t off;          // byte offset of the column in this lane's SLOT of the pass whose weights are requested next
    int n;                 // entries of that pass (wave-uniform)
    uint64_t starts;       // where the groups of that pass start
    uint32_t chunk;        // byte offset of the chunk of the lane's candidate of that pass, of the pass's last entry where it takes none
    int j;                 // group of the lane's entry inside that pass, or 4: not part of it
    uint16_t xraw[BATCH];  // its x
};

// Deals the candidates kk (-1 past the slice) and notes in h what the pass's loads and products need, but its x.  Lanes that take none point at the
// pass's last column (a line that is fetched anyway; the first column of all in a pass without entries) and carry x = 0.
template <int GROUPS, int BATCH>
__device__ __forceinline__ Deal deal_columns(PassHead<BATCH> &h, int kk, int log2g, uint32_t chunk_b, int lane) {
    const int g = kk >> log2g;
    const Deal d = deal_groups<GROUPS>(kk, g, lane);
    const int k_last = __builtin_amdgcn_readlane(kk, d.n - 1);       // (no entries: lane 63)
    const uint32_t k = (uint32_t)(d.take ? kk : (k_last < 0 ? 0 : k_last));
    h.chunk = (k >> log2g) * chunk_b;
    h.off = slot_order(h.chunk + (k & ((1u << log2g) - 1u)) * kColBytes, lane);
    h.n = d.n;
    h.starts = d.starts;
    h.j = d.take ? d.j : 4;
    return d;
}

// The scales of the lane's 4 rows in each group of the pass; behind its last one, that one's.  (They meet sums of zero, which an infinite scale makes NaN: so
// no other group's, where a row whose scale is infinite would have been infinite.)
template <int BATCH, int GROUPS>
__device__ __forceinline__ void load_scales(const uint8_t *row_base, uint32_t out4, const PassHead<BATCH> &h, u32x2 (&sc)[GROUPS]) {
    if (GROUPS == 1) {           // the group of the pass's first entry
        sc[0] = *reinterpret_cast<const u32x2 *>(row_base + (size_t)((uint32_t)__builtin_amdgcn_readfirstlane((int)h.chunk) + out4 * 8u));
        return;
    }
    uint64_t left = h.starts;
#pragma unroll
    for (int i = 0; i < GROUPS; ++i) {
        int at;      // the first start that is left, or -1, which v_readlane takes as lane 63: the last group's, whether it takes an entry or not
        asm("s_ff1_i32_b64 %0, %1\n\ts_bitset0_b64 %1, %0" : "=&s"(at), "+s"(left));
        const uint32_t chunk = (uint32_t)__builtin_amdgcn_readlane((int)h.chunk, at);
        sc[i] = *reinterpret_cast<const u32x2 *>(row_base + (size_t)(chunk + out4 * 8u));
    }
}

// The passes of a wavefront's slice, at least one.  head(p) is the HEAD of the pass that starts at entry p: it fills h, requests what
// later passes need and returns where the next pass starts; more(p) tells whether there is one.  One buffer of weights, refilled
// half by half as a pass is multiplied.  EMPTY: a pass may have no entries; its scales, which may be those of a group whose columns
// are all dropped, are then not applied (infinite ones times its sums, which are zero, would be NaN).  A branch around the adds: one launch, one
// and two rows, 0.2 % slower on average than without the test, 3 and 4 rows as fast; zeroes in place of the scales cost 0.5 and 0.2 %.
// FULL: nearly all passes are full, and their products are not worth a branch per sixteen entries (dense 5120 x 5120 6.18 us without, 6.26 with).
// first_requested and first_here: what is done, and where the timeline build stamps, when the first pass is requested.
template <int BATCH, int GROUPS, bool EMPTY, bool FULL, class Head, class More, class Stamp2, class Stamp3>
__device__ __forceinline__ void run_passes(StagedX &staged, const uint8_t *row_base, int lane, uint32_t n8, uint32_t out4,
                                           int part, int pos, PassHead<BATCH> &h, Head head, More more, Stamp2 first_requested,
                                           Stamp3 first_here, float (&acc)[BATCH][4]) {
    const uint8_t *columns = row_base + kScaleBytes;
    u32x2 w[16], sc[GROUPS];
    f32x4 d[4];
    uint32_t sign = part & 1 ? kSignOfX : 0u;
    pos = head(pos);
    load_columns<0, 16>(columns, h.off, n8, w);
    load_scales<BATCH, GROUPS>(row_base, out4, h, sc);
    const ReadsX rx(staged, lane);
    if (GROUPS == 1) clear_x(staged, lane);
    auto first_half = [&](int n) {
        quarter_pass<0>(w, rx, d);
        if (FULL || n > 16) quarter_pass<1>(w, rx, d);
    };
    auto second_half = [&](int n) {
        if (n > 32) {
            quarter_pass<2>(w, rx, d);
            if (FULL || n > 48) quarter_pass<3>(w, rx, d);
        }
    };
    first_requested();
    first_here();
    while (more(pos)) {
        stage_x<BATCH, GROUPS>(staged, lane, h.j, sign, h.xraw);
        const int n = h.n;
        pos = head(pos);
        keep_order();
        start_products(rx, d);
        first_half(n);
        keep_order();
        load_columns<0, 8>(columns, h.off, n8, w);
        keep_order();
        second_half(n);
        keep_order();
        load_columns<8, 16>(columns, h.off, n8, w);
        keep_order();
        if (!EMPTY || n > 0) {
            add_scaled<BATCH, GROUPS>(d, sc, acc);
            sign ^= kSignOfX;
        }
        load_scales<BATCH, GROUPS>(row_base, out4, h, sc);
        keep_order();
    }
    stage_x<BATCH, GROUPS>(staged, lane, h.j, sign, h.xraw);
    start_products(rx, d);
    first_half(h.n);
    second_half(h.n);
    if (!EMPTY || h.n > 0) add_scaled<BATCH, GROUPS>(d, sc, acc);
    else sign ^= kSignOfX;       // the sums still have the sign of the pass before
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
#pragma unroll
        for (int p = 0; p < 4; ++p) acc[b][p] = as_float(as_u32(acc[b][p]) ^ (sign << 16));
}

}  // namespace spqt
#endif
