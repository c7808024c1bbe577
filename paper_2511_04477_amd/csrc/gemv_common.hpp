// Device helpers shared by the GEMV kernels: the int4 multiply step and the transposing lane folds of the
// column-block kernels, the placement of workgroups, and the exchange of partial sums between the workgroups of a
// block-row.  Not part of the C ABI.
#ifndef SPQT_GEMV_COMMON_HPP
#define SPQT_GEMV_COMMON_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "split.hpp"

namespace spqt {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kPassCols = 64;                  // most columns one pass covers
constexpr float kTwo24 = 16777216.0f;          // 2^24: undoes the fp16 subnormal exponent
constexpr int kHalfOutputBit = 1 << 30;        // in the kernels' M argument: y is fp16, not fp32
constexpr int kOwnSetsBit = 1 << 29;           // in the kernels' M argument: every activation row keeps its own set
constexpr int kGroup64Bit = 1 << 28;           // in the kernels' M argument: quantization groups of 64 columns, not 128
constexpr int kRowsMask = (1 << 25) - 1;       // the bits of that argument that hold M (M <= 2^24)
#ifdef SPQT_TEST_GIVE_UP
// Test build (libspqt_giveup.so): the producers publish nothing and the reducer's wait is a handful of polls, so
// the give-up path of combine_block_row runs on every launch with several workgroups per block-row - and every
// kernel still ends normally.
constexpr int kMaxPolls = 4;
constexpr bool kMuteProducers = true;
#else
constexpr int kMaxPolls = 1 << 18;             // bound on the reducer's wait for one batch of partials
constexpr bool kMuteProducers = false;
#endif
constexpr int kHandOverPolls = 1 << 10;        // polls (about 1 ms) after which the reducer of a spread block-row hands over
#ifdef SPQT_TEST_HAND_OVER
// Test build (libspqt_handover.so): it hands over instead of waiting for the last of its words.
constexpr bool kAlwaysHandOver = true;
#else
constexpr bool kAlwaysHandOver = false;
#endif

// Per-wavefront wall-clock stamps for the timeline build (-DSPQT_TIMELINE=1, libspqt_timeline.so): every
// wavefront records when it started (0), knew its share of the list (1), had issued its first pass (2),
// had that pass's weights (3, with a forced wait that the product build does not have), left its loop (4),
// passed the workgroup's LDS reduction (5) and finished (6); word 7 tells whether it belongs to the
// reducing workgroup and where it ran.  The product build compiles all of it away.
#ifdef SPQT_TIMELINE
static __device__ unsigned long long *spqt_tl_buf = nullptr;   // one per translation unit, set by its setter
#define SPQT_TL_BEGIN() unsigned long long tl_[8] = {0, 0, 0, 0, 0, 0, 0, 0}; tl_[0] = wall_clock64()
#define SPQT_TL(i) tl_[i] = wall_clock64()
#define SPQT_TL_WAIT(i) do { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); tl_[i] = wall_clock64(); } while (0)
#define SPQT_TL_END(WAVES_, wave_, lane_, reducer_)                                                              \
    do {                                                                                                         \
        tl_[6] = wall_clock64();                                                                                 \
        if (spqt_tl_buf && (lane_) == 0) {                                                                       \
            unsigned long long *d_ = spqt_tl_buf + ((size_t)blockIdx.x * (WAVES_) + (wave_)) * 8;                \
            for (int i_ = 0; i_ < 7; ++i_) d_[i_] = tl_[i_];                                                     \
            d_[7] = (unsigned long long)((reducer_) ? 1 : 0) |                                                   \
                    ((unsigned long long)__builtin_amdgcn_s_getreg(63492) << 8) |        /* HW_ID */             \
                    ((unsigned long long)(__builtin_amdgcn_s_getreg(63508) & 15) << 40); /* XCC_ID */            \
        }                                                                                                        \
    } while (0)
#define SPQT_TL_SETTER(name)                                                                          \
    extern "C" int name(void *p) { return (int)hipMemcpyToSymbol(HIP_SYMBOL(spqt_tl_buf), &p, sizeof(p)); }
#else
#define SPQT_TL_BEGIN()
#define SPQT_TL(i)
#define SPQT_TL_WAIT(i)
#define SPQT_TL_END(WAVES_, wave_, lane_, reducer_)
#define SPQT_TL_SETTER(name)
#endif

__device__ __forceinline__ float half_bits_to_float(uint32_t h16) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h16);
}

// Bit casts go through by-value parameters on purpose: __builtin_bit_cast applied directly
// to a vector-element expression (v.y, v[i]) reads the vector's first element instead.
__device__ __forceinline__ float as_float(uint32_t bits) { return __builtin_bit_cast(float, bits); }
__device__ __forceinline__ uint32_t as_u32(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ f16x2 as_f16x2(uint32_t bits) { return __builtin_bit_cast(f16x2, bits); }

// Eight codes of one dword, nibble i = row 8d + i of the lane's 32 rows, times x: a nibble at bits 0..3 of a half is the subnormal
// n * 2^-24, one at bits 4..7 n * 2^-20 (the smallest product of a code with x * scale is 2^-72); true_rows() undoes that once per output.
__device__ __forceinline__ void fma_codes(uint32_t w, float x, float *acc) {
    const uint32_t w8 = w >> 8;
    const f16x2 a = as_f16x2(w & 0x000F000Fu);    // nibbles 0, 4
    const f16x2 b = as_f16x2(w & 0x00F000F0u);    // nibbles 1, 5
    const f16x2 c = as_f16x2(w8 & 0x000F000Fu);   // nibbles 2, 6
    const f16x2 d = as_f16x2(w8 & 0x00F000F0u);   // nibbles 3, 7
    acc[0] = __builtin_fmaf((float)a.x, x, acc[0]);
    acc[4] = __builtin_fmaf((float)a.y, x, acc[4]);
    acc[1] = __builtin_fmaf((float)b.x, x, acc[1]);
    acc[5] = __builtin_fmaf((float)b.y, x, acc[5]);
    acc[2] = __builtin_fmaf((float)c.x, x, acc[2]);
    acc[6] = __builtin_fmaf((float)c.y, x, acc[6]);
    acc[3] = __builtin_fmaf((float)d.x, x, acc[3]);
    acc[7] = __builtin_fmaf((float)d.y, x, acc[7]);
}

__device__ __forceinline__ void fma_step(u32x4 w, float x, float *acc) {
    fma_codes(w.x, x, acc + 0);
    fma_codes(w.y, x, acc + 8);
    fma_codes(w.z, x, acc + 16);
    fma_codes(w.w, x, acc + 24);
}

// Four adjacent rows of fma_codes (after the fold over the lanes), less the bias.
__device__ __forceinline__ f32x4 true_rows(const float (&r)[4], float bias) {
    constexpr float kTwo20 = kTwo24 / 16.0f;
    return f32x4{__builtin_fmaf(r[0], kTwo24, -bias), __builtin_fmaf(r[1], kTwo20, -bias), __builtin_fmaf(r[2], kTwo24, -bias),
                 __builtin_fmaf(r[3], kTwo20, -bias)};
}

// Element i of an array in global memory, with a 32-bit byte offset (the arrays that are read so are far smaller than 4 GB).
template <class V>
__device__ __forceinline__ const V *element(const V *base, uint32_t i) {
    return reinterpret_cast<const V *>(reinterpret_cast<const char *>(base) + (size_t)(i * (uint32_t)sizeof(V)));
}

// Keeps the compiler from moving instructions across: it would gather requests behind products, or products before requests.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }

// The three levels of the column fold are written as asm blocks: the lane swaps work in place
// on both of their registers (no copies), and the wait states a swap or DPP read needs after a
// VALU write of its operand are paid once per block instead of once per instruction.

// Level 1, lane pairs (l, l^8) inside every row of 16 lanes: afterwards lanes with bit 3 clear
// hold a summed over the pair, lanes with bit 3 set hold b summed over the pair - in b's
// register.  Two bank-masked DPP adds per (a, b).
#define SPQT_FOLD8(B, A)                                                              \
    "v_add_f32_dpp " B ", " B ", " B " row_ror:8 row_mask:0xf bank_mask:0xc\n\t"      \
    "v_add_f32_dpp " B ", " A ", " A " row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
__device__ __forceinline__ void fold8_x8(const float *a, float *b) {
    asm volatile("s_nop 1\n\t" SPQT_FOLD8("%0", "%8") SPQT_FOLD8("%1", "%9") SPQT_FOLD8("%2", "%10")
                     SPQT_FOLD8("%3", "%11") SPQT_FOLD8("%4", "%12") SPQT_FOLD8("%5", "%13")
                         SPQT_FOLD8("%6", "%14") SPQT_FOLD8("%7", "%15")
                 : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7])
                 : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]));
}

// Level 2, lane pairs (l, l^16): v_permlane16_swap exchanges the odd rows of its first operand
// with the even rows of its second, so a + b afterwards is, in lanes with bit 4 clear, the old a
// summed over the pair and, in the others, the old b summed over the pair.
__device__ __forceinline__ void swap16_x8(float *a, float *b) {
    asm volatile("s_nop 1\n\t"
                 "v_permlane16_swap_b32 %0, %8\n\tv_permlane16_swap_b32 %1, %9\n\t"
                 "v_permlane16_swap_b32 %2, %10\n\tv_permlane16_swap_b32 %3, %11\n\t"
                 "v_permlane16_swap_b32 %4, %12\n\tv_permlane16_swap_b32 %5, %13\n\t"
                 "v_permlane16_swap_b32 %6, %14\n\tv_permlane16_swap_b32 %7, %15"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]),
                   "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7]));
}
// Level 3, lane pairs (l, l^32), same idea with the two halves of the wave.
__device__ __forceinline__ void swap32_x4(float *a, float *b) {
    asm volatile("s_nop 1\n\t"
                 "v_permlane32_swap_b32 %0, %4\n\tv_permlane32_swap_b32 %1, %5\n\t"
                 "v_permlane32_swap_b32 %2, %6\n\tv_permlane32_swap_b32 %3, %7"
                 : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
}
__device__ __forceinline__ float fold16(float a, float b) {
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return a + b;
}
__device__ __forceinline__ float fold32(float a, float b) {
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return a + b;
}

// Fold the 32 accumulators of the 8 lanes that read the same rows (lanes seg, seg+8, ...,
// seg+56), halving the number of live values at each of the three levels.  Lane (cg, seg)
// ends with the complete sums of rows 32 seg + 4 rev(cg) + j, j = 0..3, where rev reverses
// the three bits of cg (level 1 splits on lane bit 3, level 2 on bit 4, level 3 on bit 5).
// acc is clobbered.
__device__ __forceinline__ void fold_columns(float *acc, float *out4) {
    fold8_x8(acc + 0, acc + 16);      // pairs (i, i+16), i = 0..7   -> acc[16..23]
    fold8_x8(acc + 8, acc + 24);      // pairs (i, i+16), i = 8..15  -> acc[24..31]
    swap16_x8(acc + 16, acc + 24);    // pairs (16+i, 24+i)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = acc[16 + i] + acc[24 + i];
    swap32_x4(acc + 0, acc + 4);      // pairs (i, 4+i)
#pragma unroll
    for (int i = 0; i < 4; ++i) out4[i] = acc[i] + acc[4 + i];
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return as_float(__builtin_amdgcn_update_dpp(0u, as_u32(v), CTRL, 0xf, 0xf, false));
}

// Sum over the 8 lanes that read the same rows of a column run (lanes seg, seg + 8, ..., seg + 56).
__device__ __forceinline__ float sum_over_columns(float v) {
    v += dpp_move<0x128>(v);   // row_ror:8 - the lane 8 further inside the row of 16
    v = fold16(v, v);
    v = fold32(v, v);
    return v;
}

// The one-launch kernel for one activation row: list built in the kernel, even shares (gemv_bal.hip).
hipError_t launch_gemv_bal(int waves, int grid, hipStream_t stream, const uint8_t *packed, const uint16_t *x, float thr,
                           float *y, uint32_t *ws, int K, int S, int T, int m_and_flags);

// The index-list and dense kernels (gemv_list.hip); idx == nullptr: dense.  one_group: passes of one quantization group.
struct ListLaunch {
    const uint8_t *packed;
    const uint16_t *x;
    const int32_t *idx, *count;
    float *y;
    uint32_t *ws;
    int K, S, T, m_and_flags;
};
hipError_t launch_gemv_list(int waves, int batch, bool one_group, int grid, hipStream_t stream, const ListLaunch &a);

// The order of the kernels' arguments: what a wavefront needs before it can request anything comes first.  The first 14 dwords of
// the arguments are in scalar registers when a wavefront starts (-amdgpu-kernarg-preload-count in the build), the rest is a
// load away; with that, and products with an inverse from the host in place of five divisions before the first request, a
// launch takes 0.2 to 0.5 us less (gather + GEMV where there is a list, us: 4096 x 4096 at 50 % 7.78 / 7.46, column blocks 8.11 / 7.60;
// dense 5120 x 5120 7.32 / 6.94; one launch, 11008 x 4096 at 40 % 8.00 / 7.70).

// Combine the S workgroups of block-row t (paper Section 4.2.2: the partial sums of the
// threadgroups that share a superblock row are reduced once at the end, without atomics on y).
// `red` holds this workgroup's [WAVES][BATCH][ROWS] partial sums in LDS (already synchronised);
// ROWS is the height of a block-row (256 for the 4-bit layouts).
// Every workgroup but the last (s == S-1) publishes its ROWS partial sums as 32-bit words with device-scope stores
// (two adjacent rows per store where a thread owns more than one).  A word is the sum's bits, +0 written as -0, and 0 means "not
// there yet".  The last workgroup adds the others' words in index order, polling until none is 0, then its own sums, writes y, and stores
// zero back into every word it consumed - so between calls the exchange area is all zeros whatever M, launch shape or kernel
// the calls had, and a word that is not 0 is always one of THIS call.  (A tag beside every value would double the bytes:
// four activation rows, 1024 x 4096, 16 workgroups per block-row: 9.8 us with tagged 64-bit words, 7.4 without;
// one row, 4096 x 4096: 5.6 and 5.2.)
// What bounds it: a store's way to where the other XCDs see it and a load's way back (0.4 to 0.5 us), and the instructions of the one
// wavefront per SIMD before and after, 2 ns each.  So the words to load are counted in fours (6 workgroups loaded 16 where 5 are real), a
// word is added as it is, the poison flag comes with the first words and not before them, and the words are cleared 16 bytes per lane with
// plain stores, which are acknowledged sooner than device-scope ones (nobody looks at them before the launch ends).  Before / now (us):
// list at 50 % 4096 x 4096 4.95 / 4.72, 14336 x 4096 6.95 / 6.75, 4096 x 14336 7.20 / 6.99, one launch at 40 % 4096 x 11008 7.22 / 6.94, dense
// 5120 x 5120 6.78 / 6.58, 4 rows 8192 x 28672 at 70 % 25.6 / 25.1, 2-bit 4096 x 4096 6.05 / 5.93; block-rows that are spread gain less (1024 x 4096
// 4.56 / 4.47).
//
// Why the wait ends.  A whole block-row has all its workgroups on one XCD, where they are dispatched in index order: the
// reducer has the highest index, so everything it waits for is running or finished.  The workgroups of a SPREAD block-row
// (block_of) are on several XCDs, which take their shares of a launch independently: a kernel of another stream may hold
// one XCD for any length of time while the reducer already runs on another.  There a reducer's wavefront that has polled
// kHandOverPolls times hands its values over: it publishes its own sums too, in the slot that is otherwise unused, and
// does not wait.  A producer's wavefront of a spread block-row looks at that slot once its own words are out.  A thread
// exchanges words only with the threads of its own number, and whichever of them publishes last finds all words there and
// does the sum, in the same order; should several find them, the one that takes the reducer's word out does.  (The look is
// a round trip at the end of producers only: 1024 x 4096 to 5120 x 13824 take 0 to 0.1 us longer.  A counter of arrivals,
// shared by the wavefronts of a launch, took 0.7 to 2.3 us.)
// All waits are bounded anyway, and a give-up poisons y with NaN instead of hanging and raises the workspace's poison flag
// (word 0 of its head): a late word of the abandoned call could otherwise be taken for a later call's, so from
// then on every call on that workspace yields NaN until spqt_workspace_init clears it.
__device__ __forceinline__ uint32_t exchange_word(float v) {
    const uint32_t w = as_u32(v);
    return w ? w : 0x80000000u;
}
// Keeps the computation of a value where it stands: the compiler would move it down to its use, behind a wait.  (No instruction.)
template <class V>
__device__ __forceinline__ void compute_here(V &v) { asm volatile("" : "+v"(v)); }
// The same for a pointer to global memory in scalar registers.
template <class V>
__device__ __forceinline__ void read_here(V *&p) {
    uint64_t bits = (uint64_t)p;
    asm volatile("" : "+s"(bits));
    p = (V *)(__attribute__((address_space(1))) V *)bits;
}

// Where a workgroup's outputs go.  read_now() comes once the first weights are requested: the kernel's last arguments are not in registers when
// it starts, and reading them where they are used puts a memory access on the way to the exchange.
template <int OUT>
struct Outputs {               // OUT: values of a workgroup
    float *y;
    uint32_t *ws, *slots, *mine;    // the workspace, the exchange words of the block-row, and those of this workgroup
    int M, s, S, t;
    bool y_half, spread, reducer;
    // one kernel argument carries M (<= 2^24) and the flags; the build with silent producers is for give-ups only
    __device__ __forceinline__ Outputs(int t_, int s_, int S_, int T, uint32_t *ws_, float *y_, int m_and_flags)
        : y(y_), ws(ws_), slots(nullptr), mine(nullptr), M(m_and_flags & kRowsMask), s(s_), S(S_), t(t_),
          y_half((m_and_flags & kHalfOutputBit) != 0), spread(is_spread(t_, T) && !kMuteProducers), reducer(S_ > 1 && s_ == S_ - 1) {}
    __device__ __forceinline__ void read_now() {
        read_here(y);
        read_here(ws);
        slots = ws + kWorkspaceHead / 4 + (size_t)((uint32_t)t * (uint32_t)S) * OUT;
        mine = slots + (size_t)(uint32_t)s * OUT;
        read_here(slots);
        read_here(mine);
    }
};

template <int WAVES, int BATCH, int ROWS = kTileRows>
__device__ __forceinline__ void combine_block_row(const float *red, int tid, const Outputs<BATCH * ROWS> &o) {
    constexpr int kOut = BATCH * ROWS;           // values one workgroup contributes: [BATCH][ROWS]
    constexpr int kThreads = WAVES * 64;
    constexpr int kVals = kOut > kThreads ? 2 : 1;     // adjacent values a thread moves at once: 64-bit or 32-bit accesses
    typedef std::conditional_t<kVals == 2, unsigned long long, uint32_t> Word;
    constexpr int kUnits = kOut / kVals;         // unit i = values kVals i ..
    constexpr int kPerThread = (kUnits + kThreads - 1) / kThreads;
    // A thread that owns several units handles 2 of them together, so that the reducer's loads for
    // all of them are in flight at once (one round trip instead of one per unit).
    constexpr int kTogether = kPerThread < 2 ? kPerThread : 2;
    const int S = o.S;
    Word *slots = reinterpret_cast<Word *>(o.slots);    // [S][kUnits]; S - 1: handed over
    for (int i0 = tid; kUnits == kThreads || i0 < kUnits; i0 += kTogether * kThreads) {
        uint32_t at[kTogether];
        float sum[kTogether][kVals];
#pragma unroll
        for (int i = 0; i < kTogether; ++i) {
            at[i] = (uint32_t)(i0 + i * kThreads < kUnits ? i0 + i * kThreads : i0);
#pragma unroll
            for (int q = 0; q < kVals; ++q) {
                sum[i][q] = red[kVals * at[i] + q];
#pragma unroll
                for (int w2 = 1; w2 < WAVES; ++w2) sum[i][q] += red[w2 * kOut + kVals * at[i] + q];
            }
        }
        // fp32 output, or the same value rounded to fp16 (nearest even) when the caller asked for it;
        // rows past M are the last block-row's zero padding
        uint32_t y_at[kTogether];                // element number, less than 2^26
        int rows_left[kTogether];
#pragma unroll
        for (int i = 0; i < kTogether; ++i) {
            const int r = (int)(kVals * at[i]), row = o.t * ROWS + r % ROWS;
            y_at[i] = (uint32_t)((r / ROWS) * o.M + row);
            rows_left[i] = o.M - row;
        }
        auto store_y = [&](int i, int q, float v) {
            if (q < rows_left[i]) {
                if (o.y_half) reinterpret_cast<_Float16 *>(o.y)[y_at[i] + (uint32_t)q] = (_Float16)v;
                else o.y[y_at[i] + (uint32_t)q] = v;
            }
        };
        auto word_of = [&](const float (&values)[kVals]) -> Word {
            Word word = exchange_word(values[0]);
            if (kVals == 2) word |= (Word)((unsigned long long)exchange_word(values[kVals - 1]) << 32);
            return word;
        };
        auto value_of = [&](Word word, int q) { return as_float((uint32_t)((unsigned long long)word >> (32 * q))); };
        auto publish = [&]() {
#pragma unroll
            for (int i = 0; i < kTogether; ++i) {
                if (i > 0 && at[i] == at[0]) continue;   // a clamped duplicate: already published
                if (kMuteProducers) continue;
                __hip_atomic_store(reinterpret_cast<Word *>(o.mine) + at[i], word_of(sum[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        };
        bool handed_over = false;                // (wave-uniform) the reducer of a spread block-row has not waited for all
        if (S == 1) {
#pragma unroll
            for (int i = 0; i < kTogether; ++i)
#pragma unroll
                for (int q = 0; q < kVals; ++q) store_y(i, q, sum[i][q]);
        } else if (!o.reducer) {
            publish();
            if (o.spread) {
                // A device-scope store has reached every XCD when it is acknowledged: of two threads that publish and then look
                // for each other's words one at least finds them.
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                Word there = 0;
#pragma unroll
                for (int i = 0; i < kTogether; ++i)
                    there |= __hip_atomic_load(slots + (size_t)((S - 1) * kUnits) + at[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                handed_over = __ballot(there != 0) != 0ull;
            }
        } else {
            const uint32_t poisoned = __hip_atomic_load(o.ws, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // comes with the first words
            float total[kTogether][kVals];
#pragma unroll
            for (int i = 0; i < kTogether; ++i) {
                compute_here(y_at[i]);
                compute_here(rows_left[i]);
#pragma unroll
                for (int q = 0; q < kVals; ++q) {
                    total[i][q] = 0.0f;
                    compute_here(sum[i][q]);
                }
            }
            bool all_here = true;                // wave-uniform
            // N partial sums; those from number SURE on may lie behind the block-row's, and then the first one's words are loaded once more: the words
            // behind are another block-row's, or nobody's, and a load of them goes past this XCD's L2 (8-bit list 3200 x 4864 7.78 / 7.64 us).
            auto collect = [&](auto count, auto sure, int p0) {
                constexpr int N = decltype(count)::value, SURE = decltype(sure)::value;
                Word v[kTogether][N];
                const bool at_once = kAlwaysHandOver && o.spread && p0 + N >= S - 1;
                const Word *from = slots + (size_t)(p0 * kUnits);
                uint32_t step[N];        // to partial sum p0 + j, or to p0 where that lies behind the block-row's
#pragma unroll
                for (int j = 0; j < N; ++j) step[j] = j < SURE || p0 + j < S - 1 ? (uint32_t)(j * kUnits) : 0u;
                int polls = 0;
                do {
                    // unconditional loads back to back, then one check
#pragma unroll
                    for (int j = 0; j < N; ++j)
#pragma unroll
                        for (int i = 0; i < kTogether; ++i)
                            v[i][j] = __hip_atomic_load(element(from, step[j] + at[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    uint32_t least = ~0u;   // one running minimum: a comparison per word costs 0.5 us here
#pragma unroll
                    for (int j = 0; j < N; ++j)
#pragma unroll
                        for (int i = 0; i < kTogether; ++i)
#pragma unroll
                            for (int q = 0; q < kVals; ++q) {
                                const uint32_t word = (uint32_t)((unsigned long long)v[i][j] >> (32 * q));
                                least = word < least ? word : least;
                            }
                    all_here = __builtin_amdgcn_ballot_w64(least == 0u) == 0ull;
                } while (!all_here && !at_once && ++polls < (o.spread ? kHandOverPolls : kMaxPolls));
                if (at_once) all_here = false;
#pragma unroll
                for (int j = 0; j < N; ++j)
#pragma unroll
                    for (int i = 0; i < kTogether; ++i)
#pragma unroll
                        for (int q = 0; q < kVals; ++q) {
                            const float f = value_of(v[i][j], q);
                            total[i][q] += j < SURE || p0 + j < S - 1 ? f : 0.0f;
                        }
            };
            typedef std::integral_constant<int, 1> One;
            if (S <= 5) collect(std::integral_constant<int, 4>{}, One{}, 0);
            else if (S <= 9) collect(std::integral_constant<int, 8>{}, std::integral_constant<int, 5>{}, 0);
            else if (S <= 13) collect(std::integral_constant<int, 12>{}, std::integral_constant<int, 9>{}, 0);
            else if (S <= 17) collect(std::integral_constant<int, 16>{}, std::integral_constant<int, 13>{}, 0);
            else
                for (int p0 = 0; p0 < S - 1 && all_here; p0 += 16) collect(std::integral_constant<int, 16>{}, One{}, p0);
            if (all_here || !o.spread) {
                if (!all_here) __hip_atomic_store(o.ws, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const bool bad = !all_here || poisoned;
#pragma unroll
                for (int i = 0; i < kTogether; ++i)
#pragma unroll
                    for (int q = 0; q < kVals; ++q) store_y(i, q, bad ? __builtin_nanf("") : total[i][q] + sum[i][q]);
                // Consumed: the words go back to zero for whatever call comes next.  A wavefront clears what its own lanes have seen, 16 bytes
                // per lane, i.e. several partial sums at a time.
                constexpr int kLanes = 64 * (int)sizeof(Word) / 16;      // lanes that cover the wavefront's words of one partial sum
#pragma unroll
                for (int i = 0; i < kTogether; ++i) {
                    if (i > 0 && at[i] == at[0]) continue;
                    u32x4 *to = reinterpret_cast<u32x4 *>(slots + (at[i] & ~63u)) + (tid & (kLanes - 1));
                    for (int p = (tid & 63) / kLanes; p < S - 1; p += 64 / kLanes) to[p * (kUnits * (int)sizeof(Word) / 16)] = u32x4{0u, 0u, 0u, 0u};
                }
            } else {
                handed_over = true;
                publish();
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        }
        if (handed_over) {
            // The sum of a handed-over block-row, by the thread that finds all words there.
#pragma unroll 1
            for (int i = 0; i < kTogether; ++i) {
                if (i > 0 && at[i] == at[0]) continue;
                Word *from = slots + at[i];
                bool all_here = true;
                for (int p = S - 1; p >= 0 && all_here; --p)
                    all_here = __hip_atomic_load(from + (size_t)(p * kUnits), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
                if (!all_here) continue;         // whoever publishes the missing word comes by here too
                const Word own = __hip_atomic_exchange(from + (size_t)((S - 1) * kUnits), (Word)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (own == 0) continue;          // another thread does it
                const uint32_t bad = __hip_atomic_load(o.ws, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                float total[kVals];
#pragma unroll
                for (int q = 0; q < kVals; ++q) total[q] = 0.0f;
#pragma unroll 1
                for (int p = 0; p < S; ++p) {
                    const Word v = p == S - 1 ? own : __hip_atomic_load(from + (size_t)(p * kUnits), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int q = 0; q < kVals; ++q) total[q] += value_of(v, q);
                    if (p < S - 1) __hip_atomic_store(from + (size_t)(p * kUnits), (Word)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int q = 0; q < kVals; ++q) store_y(i, q, bad ? __builtin_nanf("") : total[q]);
            }
        }
        if (kUnits == kThreads) break;
    }
}

}  // namespace spqt
#endif
