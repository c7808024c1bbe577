// spqt_gemv_fused, one activation row: sparsity test, compaction and load-balanced GEMV in ONE launch.
//
// Paper Section 4.2.3: every simdgroup that works on a block-row gets an EVEN share of the kept-column
// list (about n_ns / (n1 * n2) columns), so the work is balanced however the kept columns are spread;
// Section 2: a column is sparse iff |x_i| < threshold.  The paper builds the list with a kernel of its
// own; here every workgroup derives what it needs of the list from x itself, which removes that
// launch and the dependent global reads count -> index entries -> weights from the GEMV's start:
//   1. COUNT.  The workgroup's wavefronts bring the whole x into LDS (loads that write LDS directly, 512
//      columns = 8 fp16 per lane at a time), threshold it and leave the kept count of every 512-column
//      step in LDS (x is at most 64 KB here and sits in L2; this is popcounts only, three steps packed in
//      one word so that one lane reduction serves three steps).
//   2. SPLIT.  Every wavefront scans the step counts (at most 128), which gives n_ns and, for its own even
//      share [n_ns * j / (S * WAVES), n_ns * (j + 1) / (S * WAVES)) of the kept columns in ascending order,
//      the step in which the share begins - the very partition the index-list kernel takes from idx.
//   3. LIST.  The wavefront compacts the steps of its share, one at a time and only as the passes need
//      them, into a ring of (column, x) pairs in LDS: an exclusive scan of the lanes' kept counts ranks the
//      kept columns, and an entry whose rank falls inside the share is written at rank - share start.
//      The next step's x is requested one refill ahead, so no pass ever waits on a dependent global read.
//   4. GEMV.  Passes over the ring exactly as gemv_list.hip forms them over idx (pass.hpp),
//      same loop, same exchange between the workgroups of a block-row; for the same launch
//      shape the two kernels perform the same arithmetic in the same order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "keep.hpp"
#include "pass.hpp"

namespace {

using namespace spqt;

constexpr int kGroups = groups_per_pass(1);
constexpr int kStepCols = 512;            // columns one wavefront step thresholds: 8 per lane
constexpr int kXsSteps = 64;              // steps of x kept in LDS: K <= 32768 (larger K: static column ranges)
constexpr int kPackSteps = 3;             // step counts packed in one 32-bit word (10 bits each, a count is <= 512)
constexpr int kRing = 1024;               // ring entries per wavefront; a refill adds at most 512 to at most 63 live ones

// Number of dropped entries among the eight fp16 values of v.
__device__ __forceinline__ int dropped_count8(u32x4 v, uint32_t c2) {
    return (int)__popc(dropped_signs(magnitude_bits(v.x), c2) | (dropped_signs(magnitude_bits(v.y), c2) >> 1) | (dropped_signs(magnitude_bits(v.z), c2) >> 2) |
                       (dropped_signs(magnitude_bits(v.w), c2) >> 3));
}
// Bit i set iff entry i of the eight fp16 values of v is KEPT.
__device__ __forceinline__ uint32_t keep_bits8(u32x4 v, uint32_t c2) {
    const uint32_t u = (dropped_signs(magnitude_bits(v.x), c2) >> 15) | (dropped_signs(magnitude_bits(v.y), c2) >> 13) | (dropped_signs(magnitude_bits(v.z), c2) >> 11) |
                       (dropped_signs(magnitude_bits(v.w), c2) >> 9);
    return ~(u | (u >> 15)) & 0xFFu;
}

// Inclusive prefix sum over the 64 lanes (Hillis-Steele with DPP row shifts, then the row totals);
// total = the sum over all lanes (wave-uniform).
__device__ __forceinline__ int wave_inclusive_scan(int v, int lane, int &total) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    // totals of the rows of 16 lanes
    const int t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31);
    const int t2 = __builtin_amdgcn_readlane(v, 47), t3 = __builtin_amdgcn_readlane(v, 63);
    const int row = lane >> 4;
    total = t0 + t1 + t2 + t3;
    return v + (row > 0 ? t0 : 0) + (row > 1 ? t1 : 0) + (row > 2 ? t2 : 0);
}
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64) void spqt_gemv_bal_kernel(
    int S, int T, int K, int M, uint32_t inv, float thr, const uint16_t *__restrict__ x, const uint8_t *__restrict__ packed,
    float *__restrict__ y, uint32_t *ws) {
    __shared__ __attribute__((aligned(16))) StagedX staged[WAVES];
    __shared__ __attribute__((aligned(16))) float red[WAVES][1][kTileRows];
    // kept columns per step: word [w][q][row of 16 lanes] holds, 10 bits each, that row's counts of the steps
    // w + WAVES * (3 q + r), r = 0..2 (the steps wavefront w thresholds, three at a time)
    __shared__ __attribute__((aligned(16))) uint32_t count_part[WAVES][(kXsSteps / WAVES + kPackSteps - 1) / kPackSteps + 1][4];
    __shared__ uint32_t ring[WAVES][kRing + 64];                                       // the wavefront's share of the list: column | x bits << 16 (+ 64 dummy entries)
    __shared__ __attribute__((aligned(16))) u32x4 xs[kXsSteps * 64];                   // x, [step][lane]

    SPQT_TL_BEGIN();
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15;       // 16-row segment of the block-row this lane reads
    const uint32_t n8 = (uint32_t)n * 8u;
    const uint32_t out4 = (uint32_t)(4 * n + (lane >> 4));    // the lane's 4 outputs: rows 4 out4 .. 4 out4 + 3
    int t, s;
    if (!block_of<WAVES>(blockIdx.x, S, T, inv, t, s)) return;
    Outputs<kTileRows> outputs(t, s, S, T, ws, y, M);

    // 1. COUNT: x into LDS, then the kept columns of every 512-column step (every workgroup does all of x).
    const int nsteps = (K + kStepCols - 1) / kStepCols;      // <= kXsSteps (checked on the host)
    const uint32_t c2 = threshold_bits(thr);
    const int my_steps = (nsteps - wave + WAVES - 1) / WAVES;             // steps wave, wave + WAVES, ...
#pragma unroll 1
    for (int i = 0; i < my_steps; ++i) {
        const int j = wave + i * WAVES;
        const int c = j * kStepCols + lane * 8;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(x + (c < K ? c : 0)),
                                         (__attribute__((address_space(3))) void *)&xs[j * 64], 16, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
    for (int q = 0; q * kPackSteps < my_steps; ++q) {
        uint32_t packed = 0;
#pragma unroll
        for (int r = 0; r < kPackSteps; ++r) {
            const int i = q * kPackSteps + r;
            const int j = wave + (i < my_steps ? i : my_steps - 1) * WAVES;
            const u32x4 v = xs[j * 64 + lane];
            const bool valid = i < my_steps && j * kStepCols + lane * 8 < K;
            packed |= (uint32_t)(valid ? 8 - dropped_count8(v, c2) : 0) << (10 * r);
        }
        // sums over the rows of 16 lanes end up in lanes 15, 31, 47, 63
        packed += __builtin_amdgcn_update_dpp(0u, packed, 0x111, 0xf, 0xf, true);   // row_shr:1
        packed += __builtin_amdgcn_update_dpp(0u, packed, 0x112, 0xf, 0xf, true);   // row_shr:2
        packed += __builtin_amdgcn_update_dpp(0u, packed, 0x114, 0xf, 0xf, true);   // row_shr:4
        packed += __builtin_amdgcn_update_dpp(0u, packed, 0x118, 0xf, 0xf, true);   // row_shr:8
        if ((lane & 15) == 15) count_part[wave][q][lane >> 4] = packed;
    }
    __syncthreads();
    SPQT_TL(1);

    // 2. SPLIT: prefix sums of the step counts; this wavefront's even share of the n_ns kept columns.
    int c0 = 0;                                                 // kept columns of step `lane`
    {
        const int j = lane < nsteps ? lane : 0;
        const int i = j / WAVES;
        const u32x4 p = *reinterpret_cast<const u32x4 *>(count_part[j % WAVES][i / kPackSteps]);
        c0 = lane < nsteps ? (int)(((p.x + p.y + p.z + p.w) >> (10 * (i % kPackSteps))) & 0x3FFu) : 0;
    }
    int n_ns;
    const int p0 = wave_inclusive_scan(c0, lane, n_ns);
    const int parts = S * WAVES;
    const int part = s * WAVES + wave;
    const Share share = share_of<WAVES>(n_ns, part, parts, inv);
    const int begin = share.begin, total = share.end - begin;             // ranks [begin, begin + total) of the kept columns

    const int log2g = M & kGroup64Bit ? 6 : 7;
    const uint32_t chunk_b = (uint32_t)(kScaleBytes + (kColBytes << log2g));
    const uint8_t *row_base = packed + (size_t)t * (size_t)(K >> log2g) * chunk_b;

    float acc[1][4] = {{0.0f, 0.0f, 0.0f, 0.0f}};   // rows 4 out4 + p of the block-row, scaled, in the products' units

    if (total > 0) {
        // the step in which rank `begin` lies, and the kept columns before that step
        int step = (int)__builtin_ctzll(__ballot(p0 > begin));
        int rank_base = __builtin_amdgcn_readlane(p0 - c0, step);
        int filled = 0;                       // entries of the share written to the ring so far

        // 3. LIST: compact one more step into the ring (entries rank - begin, for ranks inside the share).
        // Every lane writes all eight of its entries; those that are dropped or outside the share go to a
        // dummy entry behind the ring, which keeps the code free of branches.
        auto refill = [&]() {
            const u32x4 v = xs[step * 64 + lane];
            const int col0 = step * kStepCols + lane * 8;
            const uint32_t m = col0 < K ? keep_bits8(v, c2) : 0u;
            int kept_here;
            const int incl = wave_inclusive_scan((int)__popc(m), lane, kept_here);
            const int e0 = rank_base + incl - (int)__popc(m) - begin;      // entry of this lane's first kept column
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = e0 + (int)__popc(m & ((1u << i) - 1u));
                const bool ok = ((m >> i) & 1u) && (uint32_t)e < (uint32_t)total;
                const uint32_t xb = (i & 1) ? (v[i >> 1] & 0xFFFF0000u) : (v[i >> 1] << 16);
                ring[wave][ok ? (e & (kRing - 1)) : kRing + lane] = (uint32_t)(col0 + i) | xb;
            }
            rank_base += kept_here;
            const int upto_rank = rank_base - begin;
            filled = upto_rank < 0 ? 0 : (upto_rank > total ? total : upto_rank);
            ++step;
            __builtin_amdgcn_wave_barrier();
        };

        // Entry p + lane of the share: its column, or -1 past the share.  The ring must hold it: refill first.
        auto fetch_k = [&](int p, uint16_t &xk) -> int {
            const int need = p + 64 < total ? p + 64 : total;
            while (filled < need && step < nsteps) refill();
            const int e = p + lane;
            const uint32_t v = ring[wave][e & (kRing - 1)];
            xk = (uint16_t)(v >> 16);
            return e < total ? (int)(v & 0xFFFFu) : -1;
        };

        PassHead<1> h;
        auto head = [&](int p) -> int {
            const int kk = fetch_k(p, h.xraw[0]);
            const Deal d = deal_columns<kGroups>(h, kk, log2g, chunk_b, lane);
            return p + d.n;
        };
        // 4. GEMV
        run_passes<1, kGroups, false, false>(staged[wave], row_base, lane, n8, out4, part, 0, h, head, [&](int p) { return p < total; },
                               [&]() { outputs.read_now(); SPQT_TL(2); }, [&]() { SPQT_TL_WAIT(3); }, acc);
    } else {
        outputs.read_now();
    }
    SPQT_TL(4);

    reinterpret_cast<f32x4 *>(red[wave][0])[out4] = f32x4{acc[0][0] * kUnit[0], acc[0][1] * kUnit[1], acc[0][2] * kUnit[2], acc[0][3] * kUnit[3]};
    __syncthreads();
    SPQT_TL(5);
    combine_block_row<WAVES, 1>(&red[0][0][0], tid, outputs);
    SPQT_TL_END(WAVES, wave, lane, S > 1 && s == S - 1);
}

}  // namespace

namespace spqt {

SPQT_TL_SETTER(spqt_timeline_set_bal)

hipError_t launch_gemv_bal(int waves, int grid, hipStream_t stream, const uint8_t *packed, const uint16_t *x, float thr,
                           float *y, uint32_t *ws, int K, int S, int T, int m_and_flags) {
    switch (waves) {
        case 1: hipLaunchKernelGGL((spqt_gemv_bal_kernel<1>), dim3(grid), dim3(64), 0, stream, S, T, K, m_and_flags, inverse_of(S * 1), thr, x, packed, y, ws); break;
        case 2: hipLaunchKernelGGL((spqt_gemv_bal_kernel<2>), dim3(grid), dim3(128), 0, stream, S, T, K, m_and_flags, inverse_of(S * 2), thr, x, packed, y, ws); break;
        default: hipLaunchKernelGGL((spqt_gemv_bal_kernel<4>), dim3(grid), dim3(256), 0, stream, S, T, K, m_and_flags, inverse_of(S * 4), thr, x, packed, y, ws); break;
    }
    return hipGetLastError();
}

}  // namespace spqt
