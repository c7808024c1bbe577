// The GEMV over an index list (paper Section 4.2.3: every wavefront of a block-row takes an even slice of the kept-column
// list; Section 4.2.2: partial sums stay local and are combined once), and the dense GEMV, for 1..4 activation rows that
// share one pass over the weights (the list is the union of the rows' kept columns).
//
// Mapping onto gfx950 (wave64):
//   - grid = T*S workgroups of WAVES wavefronts; wavefront j = s*WAVES + w of the S*WAVES that share block-row t takes
//     idx[n_ns*j/(S*WAVES) : n_ns*(j+1)/(S*WAVES)).
//   - the slice is consumed in passes of up to 64 entries (pass.hpp).  With one activation row a pass may hold columns of
//     up to 4 quantization groups, with two rows of 2, with three or four rows of one.
//   - one buffer of weights (16 loads of 8 bytes per lane), refilled half by half as a pass is multiplied: when the products
//     of slots u < 8 are done, their registers receive the same slots of the next pass, whose HEAD (deal the entries,
//     request its x and the entries of the pass after it) has run before the products.
//   - WAVES wavefronts are combined through LDS, the S workgroups of a block-row through words in a workspace
//     (gemv_common.hpp).  No floating-point atomics, so results are reproducible.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pass.hpp"

namespace {

using namespace spqt;

template <int WAVES, bool DENSE, int BATCH, int GROUPS>
__global__ __launch_bounds__(WAVES * 64) void spqt_gemv_list_kernel(
    int S, int T, int K, int M, uint32_t inv, const int32_t *__restrict__ count, const int32_t *__restrict__ idx,
    const uint8_t *__restrict__ packed, const uint16_t *__restrict__ x, float *__restrict__ y, uint32_t *ws) {
    __shared__ __attribute__((aligned(16))) StagedX staged[WAVES];
    __shared__ __attribute__((aligned(16))) float red[WAVES][BATCH][kTileRows];

    SPQT_TL_BEGIN();
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15;       // 16-row segment of the block-row this lane reads
    const uint32_t n8 = (uint32_t)n * 8u;
    const uint32_t out4 = (uint32_t)(4 * n + (lane >> 4));    // the lane's 4 outputs: rows 4 out4 .. 4 out4 + 3
    const int n_raw = DENSE ? K : *count;      // requested first
    int t, s;
    if (!block_of<WAVES>(blockIdx.x, S, T, inv, t, s)) return;
    Outputs<BATCH * kTileRows> outputs(t, s, S, T, ws, y, M);

    // (a count outside 0..K cannot come from spqt_gather; clamping keeps a corrupt one inside idx)
    const int n_ns = n_raw < 0 ? 0 : (n_raw > K ? K : n_raw);
    SPQT_TL(1);
    const int parts = S * WAVES;
    const int part = s * WAVES + wave;
    const Share share = share_of<WAVES>(n_ns, part, parts, inv);
    const int pos = share.begin, end = share.end;
    // One activation row: a list of K entries holds every column once, so every pass takes columns 0, 1, 2, ... in its place
    // whatever order the list has.  The FIRST pass then does not wait for its entries, which takes a dependent memory
    // access off the start.
    const bool all_kept = DENSE || (BATCH == 1 && n_ns == K);

    const int log2g = M & kGroup64Bit ? 6 : 7;
    const uint32_t chunk_b = (uint32_t)(kScaleBytes + (kColBytes << log2g));
    const uint8_t *row_base = packed + (size_t)t * (size_t)(K >> log2g) * chunk_b;

    float acc[BATCH][4];   // rows 4 out4 + p of the block-row, scaled, in the products' units
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
#pragma unroll
        for (int p = 0; p < 4; ++p) acc[b][p] = 0.0f;

    if (pos < end) {
        // List entry p + lane (clamped: the load is never predicated, so the number of loads in flight is the same on every
        // path).  It is an atomic load (the same instruction) because the compiler moves a plain one down to the use of its
        // value, behind the weights, and then waits for those too.
        auto fetch_k = [&](int p) -> int {
            const int e = p + lane;
            if (DENSE) return e;
            return __hip_atomic_load(element(idx, (uint32_t)(e < n_ns ? e : n_ns - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        };

        int k_next;                // the lane's list entry for the pass whose HEAD comes next
        PassHead<BATCH> h;

        // HEAD of the pass that starts at list position p < end: deal the entries to the pass's groups, request the
        // entries of the pass after it and its x.  Returns where the pass after it starts.
        auto head = [&](int p) -> int {
            if constexpr (DENSE) {
                // Consecutive columns up to the end of their group: nothing to deal (dealt like a list's entries: 5120 x 5120 6.18 us, so 6.04;
                // 5120 x 13824 9.02 / 8.92).
                const int g = p >> log2g, in_group = p - (g << log2g), left = (1 << log2g) - in_group, rest = end - p;
                h.n = rest < left ? rest : left;
                h.n = h.n < kPassCols ? h.n : kPassCols;
                const uint32_t chunk = (uint32_t)g * chunk_b;
                const int e = slot_of(lane);
                h.chunk = chunk;
                h.off = chunk + (uint32_t)in_group * kColBytes + (e < h.n ? (uint32_t)e * kColBytes : 0u);
                h.j = lane < h.n ? 0 : 4;
#pragma unroll
                for (int b = 0; b < BATCH; ++b) h.xraw[b] = *element(x, (uint32_t)(b * K + p + (lane < h.n ? lane : 0)));
                return p + h.n;
            }
            const int kk = p + lane < end ? (BATCH == 1 && all_kept ? p + lane : k_next) : -1;
            const Deal d = deal_columns<GROUPS>(h, kk, log2g, chunk_b, lane);
            const uint32_t k_own = d.take ? (uint32_t)kk : 0u;
            k_next = fetch_k(p + d.n);
#pragma unroll
            for (int b = 0; b < BATCH; ++b) h.xraw[b] = *element(x, (uint32_t)(b * K) + k_own);
            return p + d.n;
        };
        k_next = all_kept ? pos + lane : fetch_k(pos);
        SPQT_TL_WAIT(2);
        run_passes<BATCH, GROUPS, false, DENSE>(staged[wave], row_base, lane, n8, out4, part, pos, h, head, [&](int p) { return p < end; },
                                  [&]() { outputs.read_now(); }, [&]() { SPQT_TL_WAIT(3); }, acc);
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

template <int WAVES, bool DENSE, int BATCH, int GROUPS>
void start(int grid, hipStream_t stream, const ListLaunch &a) {
    hipLaunchKernelGGL((spqt_gemv_list_kernel<WAVES, DENSE, BATCH, GROUPS>), dim3(grid), dim3(WAVES * 64), 0, stream, a.S, a.T, a.K, a.m_and_flags,
                       inverse_of(a.S * WAVES), a.count, a.idx, a.packed, a.x, a.y, a.ws);
}

// Which kernels have workgroups of 8 wavefronts: an index list with one row, and 3 and 4 rows (the callers refuse the others).
template <int WAVES>
void start_waves(int batch, bool one_group, int grid, hipStream_t stream, const ListLaunch &a) {
    const bool dense = a.idx == nullptr;
    switch (batch) {
        case 1:
            // dense shares are whole runs of columns: a pass of one group loses nothing there
            if constexpr (WAVES < 8) {
                if (dense) return start<WAVES, true, 1, 1>(grid, stream, a);
                if (one_group) return start<WAVES, false, 1, 1>(grid, stream, a);
            }
            start<WAVES, false, 1, groups_per_pass(1)>(grid, stream, a);
            break;
        case 2:
            if constexpr (WAVES < 8) {
                if (dense) start<WAVES, true, 2, 1>(grid, stream, a);
                else start<WAVES, false, 2, groups_per_pass(2)>(grid, stream, a);
            }
            break;
        case 3:
            if (dense) start<WAVES, true, 3, 1>(grid, stream, a);
            else start<WAVES, false, 3, 1>(grid, stream, a);
            break;
        default:
            if (dense) start<WAVES, true, 4, 1>(grid, stream, a);
            else start<WAVES, false, 4, 1>(grid, stream, a);
            break;
    }
}

}  // namespace

namespace spqt {

SPQT_TL_SETTER(spqt_timeline_set_list)

hipError_t launch_gemv_list(int waves, int batch, bool one_group, int grid, hipStream_t stream, const ListLaunch &a) {
    switch (waves) {
        case 1: start_waves<1>(batch, one_group, grid, stream, a); break;
        case 2: start_waves<2>(batch, one_group, grid, stream, a); break;
        case 8: start_waves<8>(batch, one_group, grid, stream, a); break;
        default: start_waves<4>(batch, one_group, grid, stream, a); break;
    }
    return hipGetLastError();
}

}  // namespace spqt
