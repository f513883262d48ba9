// Merge sort of 64-bit composites in LDS, shared by the per-tile sort and by the depth order of the
// primitives.
#ifndef LMK_GS_LDS_SORT_H
#define LMK_GS_LDS_SORT_H
#include "lmk_gs_internal.h"
#include "wave_ops.h"

namespace lmk {

// Sorts up to THREADS * ITEMS composites with a merge sort:
// each thread sorts ITEMS composites in registers (a fixed network, no memory traffic), the
// runs of 2, 4 and 8 neighbouring lanes are merged in registers too (bitonic merges with DPP
// lane exchanges), and from there the sorted runs are merged pairwise through LDS, run length
// doubling: a thread finds where its ITEMS outputs start in the two runs (merge-path binary
// search) and merges them sequentially.  Runs are stored with one padding slot per 16 elements
// so that the strided accesses of neighbouring threads spread over the LDS banks.  Instances:
// 64 threads x 2 / 4 / 8 (one wavefront per short list, which is most tiles), 512 x 4 and 8,
// 1024 x 8 and 16 (a compute unit's LDS) for long lists and the chunks of the longest; the depth order's chunks take 512 x 8 or 1024 x 4.
__device__ __forceinline__ u32 ts_slot(u32 p) { return p + (p >> 4); }

__device__ __forceinline__ void ts_cswap(u64 &a, u64 &b)
{
    const u64 lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo; b = hi;
}

// ITEMS outputs, starting at output `diag`, of the merge of the sorted runs s[a0, a1) and s[a1, b1)
template <u32 ITEMS>
__device__ __forceinline__ void merge_from_lds(const u64 *s, u32 a0, u32 a1, u32 b1, u32 diag, u64 (&e)[ITEMS])
{
    const u32 lenA = a1 - a0, lenB = b1 - a1;
    u32 l0 = diag > lenB ? diag - lenB : 0, h0 = diag < lenA ? diag : lenA;
    while (l0 < h0) {
        const u32 mid = (l0 + h0) >> 1;
        if (s[ts_slot(a0 + mid)] < s[ts_slot(a1 + diag - 1 - mid)]) l0 = mid + 1; else h0 = mid;
    }
    u32 i = a0 + l0, j = a1 + (diag - l0);
    u64 ka = i < a1 ? s[ts_slot(i)] : ~0ull;
    u64 kb = j < b1 ? s[ts_slot(j)] : ~0ull;
    // Straight-line steps, selects only: an exhausted run shows the maximum value, which also is
    // what the padding holds, so "A first unless B is smaller" needs no bounds in the comparison
    // (a tie is between padding values, where the side does not matter).  The one LDS read per
    // step is not branched around: when the run has just been used up it reads slot 0 and the
    // value is dropped.
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k) {
        const bool takeA = ka <= kb;
        e[k] = takeA ? ka : kb;
        const u32 next = (takeA ? i : j) + 1u;
        const u32 lim = takeA ? a1 : b1;
        const bool more = next < lim;
        const u32 at = more ? next : 0u;
        const u64 v = s[ts_slot(at)];
        const u64 nv = more ? v : ~0ull;
        i = takeA ? next : i;
        j = takeA ? j : next;
        ka = takeA ? nv : ka;
        kb = takeA ? kb : nv;
    }
}

// The first three merge rounds need no LDS: the runs of 2, 4 and 8 neighbouring lanes are merged
// with a bitonic merge network whose lane exchanges are DPP moves (mirror within 2 / 4 / 8
// lanes for the first, "flip" stage, lane xor 1 / 2 for the half-cleaners that follow).
template <int CTRL>
__device__ __forceinline__ u64 ts_dpp(u64 v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(u32)v, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u32)(v >> 32), CTRL, 0xf, 0xf, true);
    return ((u64)(u32)hi << 32) | (u64)(u32)lo;
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;            // quad_perm [1,0,3,2], [2,3,0,1]
constexpr int kDppMirror4 = 0x1B, kDppMirror8 = 0x141;     // quad_perm [3,2,1,0], row_half_mirror

// one stage across lanes: element k meets element k (FLIP: ITEMS - 1 - k) of the partner lane;
// the lower lane of the pair keeps the smaller value
template <int CTRL, bool FLIP, u32 ITEMS>
__device__ __forceinline__ void ts_lane_stage(u64 (&e)[ITEMS], bool upper)
{
    u64 p[ITEMS];
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k) p[k] = ts_dpp<CTRL>(e[FLIP ? ITEMS - 1 - k : k]);
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k) {
        const bool mine = (e[k] < p[k]) != upper;           // lower keeps the smaller, upper the larger
        e[k] = mine ? e[k] : p[k];
    }
}

// a bitonic sequence of ITEMS values in registers -> ascending
template <u32 ITEMS>
__device__ __forceinline__ void ts_clean(u64 (&e)[ITEMS])
{
#pragma unroll
    for (u32 j = ITEMS >> 1; j > 0; j >>= 1) {
#pragma unroll
        for (u32 i = 0; i < ITEMS; ++i)
            if ((i & j) == 0) ts_cswap(e[i], e[i | j]);
    }
}

// What THREADS threads that work on one list wait on: a workgroup's barrier, or, for one wavefront -- which
// may be one of several in its workgroup, each with a list of its own -- only the order of its LDS accesses.
template <u32 THREADS>
__device__ __forceinline__ void team_sync()
{
    if (THREADS > kWave) {
        __syncthreads();
    } else {
        wave_fence();
    }
}
// Does any thread say so?  With team_sync; `flag` is a word of LDS, zero since before an earlier team_sync and the team's
// own for this call (__syncthreads_or has LDS of its own).
template <u32 THREADS>
__device__ __forceinline__ bool team_any(bool v, u32 *flag)
{
    if (THREADS <= kWave) return __builtin_amdgcn_ballot_w64(v) != 0ull;
    if (v) *flag = 1u;
    __syncthreads();
    return *flag != 0u;
}
template <u32 THREADS>
__device__ __forceinline__ u32 team_thread()
{
    u32 t = THREADS > kWave ? threadIdx.x : threadIdx.x & (kWave - 1u);
    asm volatile("" : "+v"(t));             // what follows from it is not kept in registers from one list to the next
    return t;
}

// n >= 1 composites load(0 .. n) to s[ts_slot(0 .. n)], ascending.  Called by the whole team; ends with its barrier.
template <u32 THREADS, u32 ITEMS, class Load>
__device__ __forceinline__ void sort_in_lds(u32 n, u64 *s, Load &&load)
{
    constexpr u32 CAP = THREADS * ITEMS;
    constexpr u32 kLaneRun = 8 * ITEMS;                     // sorted run length after the lane merges
    const u32 tid = team_thread<THREADS>();
    const u32 m = (n + ITEMS - 1) / ITEMS * ITEMS;          // elements in play: n rounded up to whole runs
    const u32 o0 = tid * ITEMS;
    const bool active = o0 < m;
    // each thread's ITEMS consecutive composites; beyond n the maximum value, which sorts to the end
    u64 e[ITEMS];
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k)
        e[k] = o0 + k < n ? load(o0 + k) : ~0ull;
    // sort the run in registers (bitonic network)
#pragma unroll
    for (u32 k = 2; k <= ITEMS; k <<= 1) {
#pragma unroll
        for (u32 j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
            for (u32 i = 0; i < ITEMS; ++i) {
                const u32 l = i ^ j;
                if (l > i) {
                    if ((i & k) == 0) ts_cswap(e[i], e[l]); else ts_cswap(e[l], e[i]);
                }
            }
        }
    }
    // runs of 2, 4, 8 lanes (every lane takes part; lanes beyond m hold the maximum value)
    ts_lane_stage<kDppXor1, true, ITEMS>(e, (tid & 1u) != 0u);
    ts_clean<ITEMS>(e);
    ts_lane_stage<kDppMirror4, true, ITEMS>(e, (tid & 2u) != 0u);
    ts_lane_stage<kDppXor1, false, ITEMS>(e, (tid & 1u) != 0u);
    ts_clean<ITEMS>(e);
    ts_lane_stage<kDppMirror8, true, ITEMS>(e, (tid & 4u) != 0u);
    ts_lane_stage<kDppXor2, false, ITEMS>(e, (tid & 2u) != 0u);
    ts_lane_stage<kDppXor1, false, ITEMS>(e, (tid & 1u) != 0u);
    ts_clean<ITEMS>(e);
    if (active) {
#pragma unroll
        for (u32 k = 0; k < ITEMS; ++k) s[ts_slot(o0 + k)] = e[k];
    }
    team_sync<THREADS>();

    for (u32 run = kLaneRun; run < m && run < CAP; run <<= 1) {
        if (active) {
            // outputs [o0, o0 + ITEMS) of the pair of runs holding them: A = [a0, a1), B = [a1, b1)
            const u32 a0 = (o0 / (2 * run)) * (2 * run);
            const u32 a1 = a0 + run < m ? a0 + run : m;
            const u32 b1 = a0 + 2 * run < m ? a0 + 2 * run : m;
            merge_from_lds<ITEMS>(s, a0, a1, b1, o0 - a0, e);
        }
        team_sync<THREADS>();
        if (active) {
#pragma unroll
            for (u32 k = 0; k < ITEMS; ++k) s[ts_slot(o0 + k)] = e[k];
        }
        team_sync<THREADS>();
    }
}

}  // namespace lmk
#endif
