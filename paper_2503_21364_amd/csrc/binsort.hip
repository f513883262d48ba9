// Stage 2: duplication of primitives into (tile | depth) keys, sort of the pairs into
// (tile, depth bits, index) order, per-tile ranges (the "depth sorting ... at the granularity of
// tiles" of Sec. 2.2; duplication with keys is the second kernel named in Sec. 4.2.1).
//
// The sorted order is total -- (tile, depth bits, primitive index) has no ties -- so it does not
// matter in which order a tile's pairs arrive in the tile's slice of the buffers: the per-tile
// sort fixes it.  The pairs are therefore written straight into their tile's slice, never
// partitioned by a sort over the tile bits: count per tile, scan, then write on a second walk.
//
//   count    one workgroup per 512 to 8192 (bin_block) consecutive primitives.  A rectangle of up to 32 tiles (nearly
//            all of them) is walked by its own lane -- binning rule 0: every tile; rule 1: the kept
//            tiles, from the bit mask the projection kernel left -- and counted per tile in LDS.  A
//            scene in spatial order puts a workgroup's pairs into few tiles, and the workgroup then
//            adds to the global per-tile counts with ONE returning atomic per tile it touched, not
//            per pair: the value returned is where its run starts inside that tile's slice.  The
//            (tile, start) list goes to memory for the emit kernel, at a place that follows from
//            the prefix sum over the workgroup pair counts which the projection stage left (a list
//            has at most one entry per pair).  Larger rectangles go to a list of their own.
//   count (large rectangles)  one wavefront per listed primitive (one workgroup beyond 2048 tiles)
//            walks its rectangle 64 tiles per step in row-major order (rule 1: with the
//            intersection test), one atomic per pair.  Lanes hold consecutive tiles, so the
//            atomics of one instruction fall into one or two cache lines and the memory side takes
//            them together (ten times the rate of scattered ones).  The close-up primitives of a
//            frame sit in a few workgroups; the list spreads them over the whole chip.
//   scan     two workgroups: the capacity check, exclusive prefix sum of the per-tile counts = the
//            per-tile ranges, a running position per tile for the listed primitives; and the tiles by
//            descending list length with the size classes of the per-tile sort.
//   emit     the same walks again.  A workgroup sets its LDS counters to range start + run start
//            for the tiles of its list and hands out positions from them.  A listed primitive
//            advances the tile's running position pair by pair, again with lane-consecutive
//            atomics, eight steps in flight.  What is written is the composite the list is
//            ordered by, depth bits << 32 | index.
//   tile sort  every tile's slice is sorted by that composite and rewritten in its final form (key = tile <<
//            32 | depth bits, value = index), in two launches: lists beyond 4096 pairs by 1024 threads with all the LDS
//            of a compute unit; the others by 512 threads, or by one wavefront up to 512 pairs.  The pairs go to buckets of
//            equal depth steps in LDS, one or two in each, and are ranked inside them; where the buckets get
//            too full (equal depths, dense clusters) the list goes through a merge sort instead.  Lists beyond 16384
//            pairs are merge-sorted in chunks of that many, then merged pairwise between the two pair buffers.
//
// Frames of many pairs per primitive are put together in another way (binsort_dense.h): where the buffers could hold such a
// frame, count and the count of large rectangles carry both ways and pick by D, and a last launch writes its lists.
//
// Integer work, bound by HBM traffic, global atomic throughput and, in the per-tile sorts, by
// LDS bandwidth and vector issue.  Atomics on one address are served one after the other (about
// 12 ns each), so nothing here funnels every workgroup through one counter.  The kernels read the
// pair count from device memory, so the host never waits for it: grids are sized from the
// caller's capacity and surplus workgroups leave at once.  If D exceeds the capacity nothing is
// emitted: every range is empty, the status word says so and D tells the caller how much room a
// retry needs.
#include <type_traits>

#include "binsort_dense.h"
#include "lds_sort.h"
#include "lmk_gs_internal.h"
#include "tile_test.h"
#include "tile_work.h"

namespace lmk {

constexpr u32 kMaskArea = 32;       // rectangles whose kept tiles the projection kernel recorded as a bit mask

// ---------------------------------------------------------------- walking a primitive's tiles
// A rectangle of up to kMaskArea tiles, walked by its own lane: f(tile id) for every tile that
// gets a pair, in row-major order.  Under binning rule 1 (TIGHT) those are the set bits of `mask`.
template <bool TIGHT, class F>
__device__ __forceinline__ void walk_small(ushort4 r, u32 area, u32 mask, u32 tiles_x, F &&f)
{
    const u32 w = (u32)r.z - (u32)r.x;
    const u32 inv_w = w ? (65536u + w - 1u) / w : 0u;       // slot / w == (slot * inv_w) >> 16 for slot < 32, w <= 32
    if (TIGHT) {
        while (mask) {
            const u32 slot = (u32)__builtin_ctz(mask);
            mask &= mask - 1u;
            const u32 row = (slot * inv_w) >> 16;
            f(((u32)r.y + row) * tiles_x + (u32)r.x + (slot - row * w));
        }
    } else {
        for (u32 slot = 0; slot < area; ++slot) {
            const u32 row = (slot * inv_w) >> 16;
            f(((u32)r.y + row) * tiles_x + (u32)r.x + (slot - row * w));
        }
    }
}

// One listed primitive, walked by a whole wavefront, 64 tiles of its rectangle per step in
// row-major order.  For every tile that gets a pair (under binning rule 1, TIGHT, every tile goes
// through the intersection test), first value = issue(tile, rank), then commit(tile, rank, value)
// -- kLargeBatch steps at a time, all their `issue` calls ahead of the first `commit`: `issue`
// starts a memory operation (a returning atomic) whose latency would otherwise be paid once per
// step, one after the other.  rank = the pair's number among those this wavefront found.
constexpr u32 kLargeBatch = 8;

// A rectangle shared by several wavefronts: wavefront `part` of `parts` takes batches part, part + parts, ...
template <bool TIGHT, class Issue, class Commit>
__device__ __forceinline__ void walk_large(ushort4 r, const float4 *__restrict__ feat_i, const ProjParams &pp,
                                           u32 lane, u32 part, u32 parts, Issue &&issue, Commit &&commit)
{
    const u32 w = (u32)r.z - (u32)r.x, area = w * ((u32)r.w - (u32)r.y);
    TileTest tt = make_tile_test(0.f, 0.f, 1.f, 0.f, 1.f, 0.f);
    if (TIGHT) {
        const float4 f0 = feat_i[0], f1 = feat_i[1];
        tt = make_tile_test(f0.x, f0.y, f0.z, f0.w, f1.x, opacity_tau(pp, f1.y));
    }
    const float inv_w = 1.0f / (float)w;
    u32 running = 0;
    for (u32 t0 = part * kWave * kLargeBatch; t0 < area; t0 += parts * kWave * kLargeBatch) {   // area > 0 implies w > 0; wave-uniform
        bool keep[kLargeBatch];
        u32 tile[kLargeBatch], rank[kLargeBatch];
        u64 value[kLargeBatch];
#pragma unroll
        for (u32 b = 0; b < kLargeBatch; ++b) {
            keep[b] = false; tile[b] = 0; rank[b] = 0;
            if (t0 + b * kWave < area) {                        // wave-uniform
                const u32 t = t0 + b * kWave + lane;
                bool k = t < area;
                u32 row = 0, col = 0;
                if (k) div_tiles(t, w, inv_w, row, col);
                const u32 tx = (u32)r.x + col, ty = (u32)r.y + row;
                if (TIGHT && k) k = tile_kept(tt, tx, ty);
                const u64 m = __builtin_amdgcn_ballot_w64(k);
                keep[b] = k;
                tile[b] = ty * pp.tiles_x + tx;
                rank[b] = running + __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
                running += (u32)__builtin_popcountll(m);
            }
        }
#pragma unroll
        for (u32 b = 0; b < kLargeBatch; ++b) value[b] = keep[b] ? issue(tile[b], rank[b]) : 0ull;
#pragma unroll
        for (u32 b = 0; b < kLargeBatch; ++b)
            if (keep[b]) commit(tile[b], rank[b], value[b]);
    }
}

// ---------------------------------------------------------------- count
// LDS_TILES > 0: the image has at most LDS_TILES tiles, rectangles of up to kMaskArea tiles are
// counted in LDS, larger ones listed.  LDS_TILES == 0 (images of more tiles): every primitive is
// listed.
// A workgroup takes bin_block() consecutive primitives, in rounds of 2048, kPer per thread (primitive
// tid + j THREADS).  What bounds these kernels is the chain of memory round trips of a
// workgroup, so the compute unit should be full of wavefronts: with 32 KB of counters four
// workgroups fit, and four workgroups of 512 threads are all the wavefronts it can hold.
constexpr u32 kRunBits = 17;             // a workgroup's pairs in one tile, minus one, fit these many bits
static_assert(kBinBlockMax <= (1u << kRunBits) && kLdsTilesLarge <= (1u << (32 - kRunBits)), "a tile and (count - 1) of a run are packed into a word");
template <u32 LDS_TILES> struct BinShape {
    static constexpr u32 kThreads = LDS_TILES == kLdsTilesSmall ? 512u : 1024u;
    static constexpr u32 kPer = 2048u / kThreads;           // primitives per thread and round
    static_assert(kBinBlockMax / kThreads <= 32u, "a bit for each of a thread's primitives");
    static constexpr u32 kWaves = kThreads / kWave;
    static constexpr u32 kRounds = LDS_TILES / kThreads;    // counters per thread
};
constexpr u32 kGiantArea = 2048;    // listed rectangles beyond this many tiles get a workgroup, not a wavefront

// Where the list of the counting workgroup whose first preprocess group is b starts: the pairs of all primitives before its own, from
// the two-level prefix sum the projection stage left (block_offsets inside a group of kScanGroup
// preprocess workgroups, plus the totals of the groups before).  Called by the whole workgroup
// ahead of a barrier; one partial sum per wavefront goes to s_part, list_first_finish adds them.
template <u32 THREADS>
__device__ __forceinline__ void list_first_start(const u64 *__restrict__ group_totals, u32 b, u64 *s_part,
                                                 u32 tid, u32 lane, u32 wv)
{
    const u32 groups_before = b / kScanGroup;
    u64 part = 0;
    for (u32 g = tid; g < groups_before; g += THREADS) part += group_totals[g];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o, 64);
    if (lane == 0) s_part[wv] = part;
}
template <u32 WAVES>
__device__ __forceinline__ u64 list_first_finish(const u64 *__restrict__ block_offsets, u32 b, const u64 *s_part)
{
    u64 first = block_offsets[b];
#pragma unroll
    for (u32 k = 0; k < WAVES; ++k) first += s_part[k];
    return first;
}

// With DenseArgs: the workgroups sort chunks of primitives by depth instead in a frame that goes the other way.
template <u32 LDS_TILES, bool TIGHT, class Dense>
__global__ __launch_bounds__(BinShape<LDS_TILES>::kThreads) void count_kernel(
    const u32 *__restrict__ tiles_touched, const ushort4 *__restrict__ rect, const u32 *__restrict__ tile_masks,
    u32 n, u32 tiles_x, u32 num_tiles, u32 *__restrict__ tile_count,
    ScratchHeader *__restrict__ header, u32 *__restrict__ big_idx,
    const u32 *__restrict__ block_sums, u32 pre_blocks,
    const u64 *__restrict__ block_offsets, const u64 *__restrict__ group_totals,
    u32 *__restrict__ bin_count, uint2 *__restrict__ list, u64 list_capacity, Dense dense)
{
    constexpr bool LDS = LDS_TILES > 0;
    constexpr u32 kThreads = BinShape<LDS_TILES>::kThreads, kPer = BinShape<LDS_TILES>::kPer;
    constexpr u32 kWaves = BinShape<LDS_TILES>::kWaves;
    constexpr u32 kRounds = LDS ? BinShape<LDS_TILES>::kRounds : 1;
    constexpr u32 kSmallMax = LDS ? kMaskArea : 0u;
    constexpr u32 kHistWords = LDS ? LDS_TILES : 1u, kSortWords = Dense::kDense ? 2u * (kSortChunk + kSortChunk / 16u) : 0u;
    __shared__ __attribute__((aligned(16))) u32 s_hist[kHistWords > kSortWords ? kHistWords : kSortWords];
    __shared__ u32 s_next;
    __shared__ u32 s_wave[kWaves][2];
    __shared__ u32 s_base[2];
    __shared__ u64 s_part[kWaves];
    bool other_way = false;
    if constexpr (Dense::kDense) other_way = header->dup_count >= dense.dense_min;
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 block = bin_block(n, num_tiles, in_order(header, n));
    const BinShare share = bin_share(blockIdx.x, block, n);
    const u32 beg = share.beg;
    if constexpr (Dense::kDense) {
        if (other_way) {                                    // the same for the whole workgroup
            sort_chunk<kThreads, TIGHT>(dense, reinterpret_cast<u64 *>(s_hist));
            return;
        }
    }
    if (share.count == 0u) return;                          // there for a chunk, or for smaller blocks
    {   // the projection stage counted the pairs of every 256 primitives: a workgroup none of whose
        // primitives was binned (culled, or a skipped voxel range) leaves without reading one
        const u32 pb = beg / kPreBlock + lane;
        static_assert(kBinBlockMax / kPreBlock <= kWave, "a lane for each");
        const bool some = lane < block / kPreBlock && pb < pre_blocks && block_sums[pb] != 0u;
        if (__builtin_amdgcn_ballot_w64(some) == 0ull) {    // the same for the whole workgroup
            if (LDS && tid == 0) bin_count[blockIdx.x] = 0;
            return;
        }
    }
    // everything that a thread needs of its primitives of a round is requested at once, a round ahead
    struct Round { u32 cnt[kPer], mask[kPer]; ushort4 r[kPer]; } next;
    auto request = [&](u32 first) {
#pragma unroll
        for (u32 j = 0; j < kPer; ++j) {
            const u32 i = first + j * kThreads + tid;
            const bool in = i - beg < share.count;
            next.cnt[j] = in ? tiles_touched[i] : 0u;
            next.r[j] = in ? rect[i] : make_ushort4(0, 0, 0, 0);
            next.mask[j] = (TIGHT && LDS && in) ? tile_masks[i] : 0u;
        }
    };
    request(beg);
    if (LDS) {
        list_first_start<kThreads>(group_totals, beg / kPreBlock, s_part, tid, lane, wv);
        for (u32 t = tid; t < num_tiles; t += kThreads) s_hist[t] = 0;
        if (tid == 0) s_next = 0;
    }
    __syncthreads();
    u32 large_bits = 0, giant_bits = 0;                     // bit k: this thread's primitive beg + k kThreads + tid goes to the list
    for (u32 first = beg, k = 0; first - beg < share.count; first += kPer * kThreads) {
        const Round now = next;
        request(first + kPer * kThreads);
#pragma unroll
        for (u32 j = 0; j < kPer; ++j, ++k) {
            const u32 area = now.cnt[j] ? ((u32)now.r[j].z - (u32)now.r[j].x) * ((u32)now.r[j].w - (u32)now.r[j].y) : 0u;
            if (LDS && area > 0u && area <= kSmallMax) {
                walk_small<TIGHT>(now.r[j], area, now.mask[j], tiles_x, [&](u32 tile) {
                    if (tile < num_tiles) atomicAdd(&s_hist[tile], 1u);     // a rectangle never leaves the grid; a corrupt one must not either
                });
            }
            if (area > kGiantArea) giant_bits |= 1u << k;
            else if (area > kSmallMax) large_bits |= 1u << k;
        }
    }
    // the lists of the other primitives (wavefront-sized rectangles from the front of big_idx,
    // workgroup-sized ones from the back): one global atomic each per workgroup that has any
    const u32 my_large = (u32)__builtin_popcount(large_bits), my_giant = (u32)__builtin_popcount(giant_bits);
    if (__syncthreads_or((my_large | my_giant) != 0u)) {    // also: every LDS count above is done
        u32 incl = my_large, incl2 = my_giant;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const u32 v = __shfl_up(incl, o, 64), v2 = __shfl_up(incl2, o, 64);
            if ((int)lane >= o) { incl += v; incl2 += v2; }
        }
        if (lane == kWave - 1) { s_wave[wv][0] = incl; s_wave[wv][1] = incl2; }
        __syncthreads();
        u32 before = 0, total = 0, before2 = 0, total2 = 0;
#pragma unroll
        for (u32 k = 0; k < kWaves; ++k) {
            const u32 w = s_wave[k][0], w2 = s_wave[k][1];
            if (k < wv) { before += w; before2 += w2; }
            total += w; total2 += w2;
        }
        if (tid == 0) {
            s_base[0] = total ? atomicAdd(&header->big_count, total) : 0u;
            s_base[1] = total2 ? atomicAdd(&header->giant_count, total2) : 0u;
        }
        __syncthreads();
        u32 slot = s_base[0] + before + incl - my_large;
        u32 slot2 = s_base[1] + before2 + incl2 - my_giant;
        // the two lists hold one entry per primitive at most, n in all, and never meet
        for (; large_bits; large_bits &= large_bits - 1u, ++slot)
            if (slot < n) big_idx[slot] = beg + (u32)__builtin_ctz(large_bits) * kThreads + tid;
        for (; giant_bits; giant_bits &= giant_bits - 1u, ++slot2)
            if (slot2 < n) big_idx[n - 1u - slot2] = beg + (u32)__builtin_ctz(giant_bits) * kThreads + tid;
    }
    if (!LDS) return;
    // The tiles this workgroup touched, compacted to the front of s_hist as tile << kRunBits | (count - 1)
    // (a workgroup holds at most kBinBlockMax primitives and a primitive has one pair per tile at most): every
    // thread first reads its counters, then, all reads done, the entries are written.
    u32 c[kRounds];
#pragma unroll
    for (u32 k = 0; k < kRounds; ++k) {
        const u32 t = k * kThreads + tid;
        c[k] = t < num_tiles ? s_hist[t] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (u32 k = 0; k < kRounds; ++k) {
        const u64 nz = __builtin_amdgcn_ballot_w64(c[k] != 0u);
        if (nz == 0ull) continue;                           // wave-uniform
        u32 at = 0;
        const int leader = (int)__builtin_ctzll(nz);
        if ((int)lane == leader) at = atomicAdd(&s_next, (u32)__builtin_popcountll(nz));
        at = __shfl(at, leader, 64);
        if (c[k] != 0u)
            s_hist[at + __builtin_amdgcn_mbcnt_hi((u32)(nz >> 32), __builtin_amdgcn_mbcnt_lo((u32)nz, 0u))] =
                ((k * kThreads + tid) << kRunBits) | ((c[k] - 1u) & ((1u << kRunBits) - 1u));
    }
    __syncthreads();
    const u32 touched = s_next;
    const u64 first = list_first_finish<kWaves>(block_offsets, beg / kPreBlock, s_part);
    if (tid == 0) bin_count[blockIdx.x] = touched;
    // one reservation per touched tile: the run of this workgroup starts where the tile's counter
    // stood; up to kFlush entries per thread with their atomics in flight together
    constexpr u32 kFlush = 4;
    for (u32 k0 = 0; k0 < touched; k0 += kFlush * kThreads) {
        u32 ent[kFlush], start[kFlush];
#pragma unroll
        for (u32 q = 0; q < kFlush; ++q) {
            const u32 k = k0 + q * kThreads + tid;
            ent[q] = k < touched ? s_hist[k] : 0u;
            start[q] = k < touched ? atomicAdd(&tile_count[ent[q] >> kRunBits], (ent[q] & ((1u << kRunBits) - 1u)) + 1u) : 0u;
        }
#pragma unroll
        for (u32 q = 0; q < kFlush; ++q) {
            const u32 k = k0 + q * kThreads + tid;
            if (k < touched && first + k < list_capacity) list[first + k] = make_uint2(ent[q] >> kRunBits, start[q]);
        }
    }
}

// Fixed grids stride over the deferred lists: the first kGiantBlocks workgroups take the
// workgroup-sized rectangles (their wavefronts share a rectangle batch by batch), the wavefronts of
// the others the wavefront-sized ones.
constexpr u32 kLargeThreads = 256, kLargeBlocks = 2048, kGiantBlocks = 1024;

// f(rectangle index, primitive index, part, parts) for every listed primitive this wavefront
// has a share of: workgroup `block` of `blocks`, THREADS threads each; the first `giant_blocks` of
// them take the list of workgroup-sized rectangles.
template <u32 THREADS, class F>
__device__ __forceinline__ void for_each_listed(const ScratchHeader *__restrict__ header, const u32 *__restrict__ big_idx,
                                                u32 n, u32 block, u32 blocks, u32 giant_blocks, u32 tid, F &&f)
{
    constexpr u32 kWaves = THREADS / kWave;
    if (block < giant_blocks) {
        u32 count = header->giant_count;
        if (count > n) count = n;                           // cannot happen: one entry per primitive at most
        for (u32 k = block; k < count; k += giant_blocks) { // uniform
            const u32 i = big_idx[n - 1u - k];
            if (i < n) f(i, tid / kWave, kWaves);
        }
    } else {
        const u32 wave = ((block - giant_blocks) * THREADS + tid) / kWave, waves = (blocks - giant_blocks) * kWaves;
        u32 count = header->big_count;
        if (count > n) count = n;
        for (u32 k = wave; k < count; k += waves) {         // wave-uniform
            const u32 i = big_idx[k];
            if (i < n) f(i, 0u, 1u);
        }
    }
}

static_assert(kLargeThreads == kDenseThreads, "the launch carries the count of both ways");
template <bool TIGHT, class Dense>
__global__ __launch_bounds__(kLargeThreads, Dense::kDense ? 6 : 1) void count_large_kernel(     // (the other way's count: 79 registers)
    const ushort4 *__restrict__ rect, const float4 *__restrict__ feat, ProjParams pp, u32 n, u32 num_tiles,
    u32 *__restrict__ large_count, const ScratchHeader *__restrict__ header, const u32 *__restrict__ big_idx,
    u32 giant_blocks, u32 blocks, u32 *__restrict__ tile_count, Dense dense)
{
    if constexpr (Dense::kDense) {
        __shared__ CountSpace s_space[kDenseWaves];
        if (header->dup_count >= dense.dense_min) {
            dense_count<TIGHT>(dense, header, tile_count, s_space);
            return;
        }
        if (blockIdx.x >= blocks) return;
    }
    const u32 lane = threadIdx.x & (kWave - 1);
    for_each_listed<kLargeThreads>(header, big_idx, n, blockIdx.x, blocks, giant_blocks, threadIdx.x,
        [&](u32 i, u32 part, u32 parts) {
            walk_large<TIGHT>(rect[i], feat + (size_t)i * (LMK_GS_FEAT_STRIDE / 4), pp, lane, part, parts,
                [&](u32 tile, u32) -> u64 { if (tile < num_tiles) atomicAdd(&large_count[tile], 1u); return 0ull; },
                [&](u32, u32, u64) {});
        });
}

// ---------------------------------------------------------------- scan + order + size classes
// Two workgroups, each of which is a chain of memory round trips and barriers rather than data, so
// they run side by side.  Both: (1) D = sum of the per-tile counts; more than the buffers hold:
// status, and every list is treated as empty from here on.  Workgroup 0: (2) tile_offsets =
// exclusive prefix sum of the counts.  Workgroup 1: (3) tile ids by descending list length, bucketed by the bit length of (length - 1), so that
// the size classes of the per-tile sort are whole buckets.  From the front of `order`:
//   classes[0]  lists longer than kHuge pairs          one workgroup of 1024 each, merges between the pair buffers
//   classes[3]  kMid + 1 .. kHuge ("long")             one workgroup of 1024
//   classes[1]  kLow + 1 .. kMid                       one workgroup of 512, eight pairs a thread
//   classes[2]  kSmallCap + 1 .. kLow                  one workgroup of 512, four pairs a thread
//   the rest                                           one wavefront each
// Within a bucket the order is whatever the atomics give -- it only decides which workgroup
// starts first, never a result.  The counters stay as they are until both workgroups are done with them; the last kernel of the
// per-tile sort leaves them zero for the next call.
// With CHUNKS (1 up to 8192 tiles, 4 up to 32768) every thread reads its eight counters of each chunk of 8192 once, all together, and
// everything else works from registers and LDS; more tiles (0) are read again for every step (32 400 tiles: 66 us so, 21 with
// four chunks).
//   classes[5]  (kDenseClass) 1 = the frame's lists come from dense_emit, sorted: nothing is emitted or sorted here
constexpr u32 kSmallThreads = 64, kSmallItems = 8, kSmallCap = kSmallThreads * kSmallItems;   // 512
constexpr u32 kLow = 2048;                                                                    // kMidThreads * kMidItems / 2
constexpr u32 kMidThreads = 512, kMidItems = 8, kMid = kMidThreads * kMidItems;               // 4096
constexpr u32 kHugeThreads = 1024, kHugeItems = 16, kHuge = kHugeThreads * kHugeItems;        // 16384
constexpr u32 kLongBlocks = 256;                            // compute units

__device__ __forceinline__ u32 length_bucket(u32 len)
{
    return len > 1u ? 32u - (u32)__builtin_clz(len - 1u) : 0u;   // len in (2^(b-1), 2^b]
}
constexpr u32 kSmallBucket = 9, kLowBucket = 11, kMidBucket = 12, kHugeBucket = 14;   // 2^9 = kSmallCap, 2^11 = kLow, 2^12 = kMid, 2^14 = kHuge

// Most tiles fall into a handful of buckets, and LDS atomics on one word are served one after
// the other: every bucket has kOrderCopies counters, picked by the low lane bits, so that the 64
// atomics of a wavefront spread over that many words.  An exclusive scan over
// [bucket][copy] turns the counts into the first slot of every (bucket, copy).  A bucket's lists that the compositing kernels
// may share between workgroups (long_list_from) come in front of its others, so that they are the first of the order.
constexpr u32 kScanThreads = 1024, kScanItems = 8;
constexpr u32 kOrderCopies = 16, kOrderBuckets = 2 * 33, kOrderCounters = kOrderBuckets * kOrderCopies;
constexpr u32 kOrderStage = 32768;
static_assert(kOrderCounters <= 2 * kScanThreads, "the counters are scanned two per thread");
constexpr u32 kScanChunk = kScanThreads * kScanItems;
static_assert(kLdsTilesSmall == kScanChunk && kLdsTilesLarge == 4u * kScanChunk && kOrderStage >= 4u * kScanChunk, "chunks of kScanItems tiles per thread");

template <u32 CHUNKS>
__global__ __launch_bounds__(kScanThreads) void tile_scan_kernel(
    const u32 *__restrict__ tile_count, const u32 *__restrict__ large_count, u32 num_tiles, u64 capacity, ScratchHeader *__restrict__ header,
    u64 *__restrict__ tile_offsets, u32 *__restrict__ tile_cursor, u64 *__restrict__ prim_offsets_if_empty,
    u32 *__restrict__ order, u32 *__restrict__ order_copy, u32 *__restrict__ classes, u64 dense_min)
{
    constexpr u32 kWaves = kScanThreads / kWave;
    // the running positions of the emit kernel are 32 bits wide: absolute where every position
    // fits (they start at the tile's range start), else relative to the range start
    const bool wide = capacity > 0xffffffffull;
    __shared__ u64 s_sum[kWaves];
    __shared__ u32 s_cnt[kOrderCounters];
    __shared__ u32 s_wave[kWaves];
    // slots are scattered and one compute unit does all the address work: the order is put
    // together in LDS and written out in whole lines (images of up to kOrderStage tiles)
    constexpr u32 kHeld = CHUNKS * kScanItems;
    constexpr bool HELD = CHUNKS > 0;
    __shared__ __attribute__((aligned(16))) u32 s_space[CHUNKS == 1u ? 2 * kScanChunk : kOrderStage];
    u32 *const s_order = s_space;
    u32 *const s_len = s_space + kScanChunk;                        // HELD: the list lengths of a chunk
    const bool staged = HELD || num_tiles <= kOrderStage;
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;

    // ---- (1) D
    // a tile's list = the runs of the counting workgroups (tile_count) followed by the pairs of
    // the listed primitives (large_count)
    u32 held[HELD ? kHeld : 1], runs[HELD ? kHeld : 1];    // HELD: list length and length of the runs of tiles j * kScanThreads + tid
    u64 part = 0;
    if constexpr (HELD) {
#pragma unroll
        for (u32 j = 0; j < kHeld; ++j) {
            const u32 t = j * kScanThreads + tid;
            runs[j] = t < num_tiles ? tile_count[t] : 0u;
            held[j] = t < num_tiles ? large_count[t] : 0u;
        }
#pragma unroll
        for (u32 j = 0; j < kHeld; ++j) {
            held[j] += runs[j];
            part += held[j];
        }
    } else {
        for (u32 t = tid; t < num_tiles; t += kScanThreads) part += (u64)tile_count[t] + large_count[t];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o, 64);
    if (lane == 0) s_sum[wv] = part;
    __syncthreads();
    u64 D = 0;
#pragma unroll
    for (u32 k = 0; k < kWaves; ++k) D += s_sum[k];
    const bool overflow = D > capacity;
    // two workgroups share the work: 0 writes D, the status and the ranges, 1 the order and the size
    // classes; both need the list lengths and D
    const bool ranges_part = blockIdx.x == 0;
    if (tid == 0 && ranges_part) {
        u32 elsewhere = 0u;
        if (dense_min != ~0ull) {                           // (else nobody asks, and the read would be a trip to memory)
            const u64 counted = header->dup_count;
            elsewhere = counted >= dense_min ? 1u : 0u;     // as the counting kernels decided
            header->counted = counted;
        }
        classes[kDenseClass] = elsewhere;
        header->dup_count = D;
        header->status = overflow ? LMK_GS_ERR_CAPACITY : LMK_GS_OK;      // of this call; the frame's earlier calls do not count
        // with no primitives nothing else writes the one-entry prefix sum over the primitives
        if (prim_offsets_if_empty) prim_offsets_if_empty[0] = 0;
    }
    if constexpr (HELD) {
#pragma unroll
        for (u32 j = 0; j < kHeld; ++j)
            if (overflow) { held[j] = 0u; runs[j] = 0u; }
    }
    __syncthreads();                           // s_sum is reused below

    // ---- (2) HELD: consecutive lanes read and write consecutive tiles, and LDS changes between that
    // and kScanItems consecutive tiles per thread (addressed in memory like that, one compute unit takes some 3.5 us for
    // the lines of the offsets alone; frame of 500 000 at 1080p, 8160 tiles: 249.0 us so, 239.5 through LDS)
    if (HELD && ranges_part) {
        u64 carry = 0;
#pragma unroll
        for (u32 chunk = 0; chunk < CHUNKS; ++chunk) {
            if (chunk * kScanChunk > num_tiles) break;
            if (chunk) __syncthreads();        // the chunk before has been written
#pragma unroll
            for (u32 j = 0; j < kScanItems; ++j) s_len[j * kScanThreads + tid] = held[HELD ? chunk * kScanItems + j : 0u];
            __syncthreads();
            const uint4 c0 = *reinterpret_cast<const uint4 *>(s_len + tid * kScanItems), c1 = *reinterpret_cast<const uint4 *>(s_len + tid * kScanItems + 4);
            const u32 c[kScanItems] = { c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w };
            u64 mine = 0;
#pragma unroll
            for (u32 j = 0; j < kScanItems; ++j) mine += c[j];
            u64 incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const u64 v = __shfl_up(incl, o, 64);
                if ((int)lane >= o) incl += v;
            }
            if (lane == kWave - 1) s_sum[wv] = incl;
            __syncthreads();                   // also: every length has been read
            u64 run = carry + incl - mine, total = 0;
#pragma unroll
            for (u32 k = 0; k < kWaves; ++k) {
                const u64 v = s_sum[k];
                if (k < wv) run += v;
                total += v;
            }
            carry += total;
            u64 *s_run = reinterpret_cast<u64 *>(s_space);
#pragma unroll
            for (u32 j = 0; j < kScanItems; ++j) { s_run[tid * kScanItems + j] = run; run += c[j]; }
            __syncthreads();
#pragma unroll
            for (u32 j = 0; j < kScanItems; ++j) {
                const u32 in = j * kScanThreads + tid, t = chunk * kScanChunk + in;
                if (t <= num_tiles) {
                    const u64 at = s_run[in];
                    tile_offsets[t] = at;
                    tile_cursor[t] = (wide ? 0u : (u32)at) + runs[HELD ? chunk * kScanItems + j : 0u];     // the listed primitives' pairs follow the runs
                }
            }
        }
        if (num_tiles == CHUNKS * kScanChunk && tid == 0) {
            tile_offsets[num_tiles] = carry;
            tile_cursor[num_tiles] = wide ? 0u : (u32)carry;
        }
        return;
    }

    // ---- (2) per-tile ranges of more tiles: kScanItems consecutive ones per thread, entry num_tiles = the end
    u64 carry = 0;
    for (u32 base = 0; !HELD && ranges_part && base <= num_tiles; base += kScanChunk) {
        const u32 t0 = base + tid * kScanItems;
        u32 c[kScanItems], runs[kScanItems];
        u64 mine = 0;
#pragma unroll
        for (u32 j = 0; j < kScanItems; ++j) {
            const bool in = !overflow && t0 + j < num_tiles;
            runs[j] = in ? tile_count[t0 + j] : 0u;
            c[j] = runs[j] + (in ? large_count[t0 + j] : 0u);
            mine += c[j];
        }
        u64 incl = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const u64 v = __shfl_up(incl, o, 64);
            if ((int)lane >= o) incl += v;
        }
        if (lane == kWave - 1) s_sum[wv] = incl;
        __syncthreads();
        u64 before = carry, total = carry;
#pragma unroll
        for (u32 k = 0; k < kWaves; ++k) {
            const u64 v = s_sum[k];
            if (k < wv) before += v;
            total += v;
        }
        u64 run = before + incl - mine;
#pragma unroll
        for (u32 j = 0; j < kScanItems; ++j) {
            if (t0 + j <= num_tiles) {
                tile_offsets[t0 + j] = run;
                tile_cursor[t0 + j] = (wide ? 0u : (u32)run) + runs[j];   // the listed primitives' pairs follow the runs
            }
            run += c[j];
        }
        carry = total;
        __syncthreads();                       // s_sum free again
    }

    if (ranges_part) return;

    // ---- (3) order and size classes.  Tile of (thread, round j): base + j * kScanThreads + tid.
    const u32 copy = tid & (kOrderCopies - 1);
    const u64 min64 = overflow || num_tiles > kSharedMaxTiles ? 0ull : long_list_from(D);
    const u32 min_long = min64 < 0xffffffffull ? (u32)min64 : 0xffffffffu;
    auto order_counter = [&](u32 len) {                                 // long lists first
        return ((32u - length_bucket(len)) * 2u + (len >= min_long ? 0u : 1u)) * kOrderCopies + copy;
    };
    for (u32 k = tid; k < kOrderCounters; k += kScanThreads) s_cnt[k] = 0;
    __syncthreads();
    // f(tile, list length) for this thread's tiles
    auto each_tile = [&](auto &&f) {
        if constexpr (HELD) {
#pragma unroll
            for (u32 j = 0; j < kHeld; ++j) {
                const u32 t = j * kScanThreads + tid;
                if (t < num_tiles) f(t, held[j]);
            }
        } else {
            for (u32 base = 0; base < num_tiles; base += kScanChunk) {
#pragma unroll
                for (u32 j = 0; j < kScanItems; ++j) {
                    const u32 t = base + j * kScanThreads + tid;
                    if (t < num_tiles) f(t, overflow ? 0u : tile_count[t] + large_count[t]);
                }
            }
        }
    };
    each_tile([&](u32, u32 len) { atomicAdd(&s_cnt[order_counter(len)], 1u); });
    __syncthreads();
    // exclusive scan of the counters, two per thread
    const u32 k0 = 2 * tid, k1 = 2 * tid + 1;
    const u32 c0 = k0 < kOrderCounters ? s_cnt[k0] : 0u, c1 = k1 < kOrderCounters ? s_cnt[k1] : 0u;
    u32 incl = c0 + c1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const u32 v = __shfl_up(incl, o, 64);
        if ((int)lane >= o) incl += v;
    }
    if (lane == kWave - 1) s_wave[wv] = incl;
    __syncthreads();
    u32 before = 0;
    for (u32 k = 0; k < wv; ++k) before += s_wave[k];
    const u32 excl = before + incl - (c0 + c1);
    if (k0 < kOrderCounters) s_cnt[k0] = excl;
    if (k1 < kOrderCounters) s_cnt[k1] = excl + c0;
    __syncthreads();
    if (tid == 0) {
        // tiles in buckets above a class limit = first slot of the first bucket at or below it
        const u32 huge = s_cnt[(32 - kHugeBucket) * 2 * kOrderCopies];
        const u32 lng = s_cnt[(32 - kMidBucket) * 2 * kOrderCopies];
        const u32 mid = s_cnt[(32 - kLowBucket) * 2 * kOrderCopies];
        const u32 low = s_cnt[(32 - kSmallBucket) * 2 * kOrderCopies];
        classes[0] = huge; classes[3] = lng - huge; classes[1] = mid - lng; classes[2] = low - mid;
    }
    __syncthreads();                           // the counters are advanced below
    each_tile([&](u32 t, u32 len) {
        const u32 slot = atomicAdd(&s_cnt[order_counter(len)], 1u);
        if (staged) {
            s_order[slot] = t;
        } else {
            order[slot] = t;
            if (order_copy) order_copy[slot] = t;
        }
    });
    if (staged) {
        __syncthreads();
        for (u32 k = tid; k < num_tiles; k += kScanThreads) {
            const u32 t = s_order[k];
            order[k] = t;
            if (order_copy) order_copy[k] = t;
        }
    }
    // the counters are left as they are: the other workgroup may still be reading them; the last
    // kernel of the per-tile sort zeroes them
}

// ---------------------------------------------------------------- emit
// Workgroups [0, bin_blocks) repeat the walk of the small rectangles of their primitives; the
// LDS counters now start at the tile's range start + the workgroup's run start and hand out
// positions.  The workgroups behind them walk the listed primitives and advance the tiles'
// running positions pair by pair.
// WIDE: positions need 64 bits (capacity of 2^32 pairs or more): LDS counters and running
// positions are then relative to the tile's range start, which is read from memory for every pair.
template <u32 LDS_TILES, bool TIGHT, bool WIDE>
__global__ __launch_bounds__(BinShape<LDS_TILES>::kThreads) void emit_kernel(
    const u32 *__restrict__ tiles_touched, const ushort4 *__restrict__ rect, const float *__restrict__ depth,
    const float4 *__restrict__ feat, const u32 *__restrict__ tile_masks, u32 n, ProjParams pp, u32 num_tiles,
    const u64 *__restrict__ tile_offsets, u32 *__restrict__ tile_cursor, const ScratchHeader *__restrict__ header,
    const u32 *__restrict__ big_idx, const u64 *__restrict__ block_offsets, const u64 *__restrict__ group_totals,
    const u32 *__restrict__ bin_count, const uint2 *__restrict__ list, u64 list_capacity,
    u32 bin_blocks, u32 giant_blocks, u64 capacity, u64 *__restrict__ keys, const u32 *__restrict__ classes)
{
    constexpr bool LDS = LDS_TILES > 0;
    constexpr u32 kThreads = BinShape<LDS_TILES>::kThreads, kPer = BinShape<LDS_TILES>::kPer;
    constexpr u32 kWaves = BinShape<LDS_TILES>::kWaves;
    __shared__ u32 s_cur[LDS ? LDS_TILES : 1];
    __shared__ u64 s_part[kWaves];
    // (here and below the flag is read together with what is needed anyway: one round trip to memory)
    const u32 elsewhere = classes[kDenseClass];             // the lists are written by dense_emit
    const int32_t status = header->status;                  // more pairs than the buffers hold: nothing is emitted
    if ((elsewhere != 0u) | (status != LMK_GS_OK)) return;
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    if (blockIdx.x >= bin_blocks) {
        for_each_listed<kThreads>(header, big_idx, n, blockIdx.x - bin_blocks, gridDim.x - bin_blocks, giant_blocks, tid,
            [&](u32 i, u32 part, u32 parts) {
                const u64 comp = ((u64)__float_as_uint(depth[i]) << 32) | (u64)i;
                walk_large<TIGHT>(rect[i], feat + (size_t)i * (LMK_GS_FEAT_STRIDE / 4), pp, lane, part, parts,
                    [&](u32 tile, u32) -> u64 {
                        if (tile >= num_tiles) return ~0ull;
                        const u32 at = atomicAdd(&tile_cursor[tile], 1u);
                        return WIDE ? tile_offsets[tile] + at : (u64)at;
                    },
                    [&](u32, u32, u64 pos) { if (pos < capacity) keys[pos] = comp; });
            });
        return;
    }
    if (!LDS) return;                                       // every primitive is on a list
    const u32 block = bin_block(n, num_tiles, in_order(header, n));
    const BinShare share = bin_share(blockIdx.x, block, n);
    if (share.count == 0u) return;
    const u32 entries = bin_count[blockIdx.x];
    if (entries == 0u) return;                              // the same for the whole workgroup
    const u32 beg = share.beg;
    list_first_start<kThreads>(group_totals, beg / kPreBlock, s_part, tid, lane, wv);
    // this thread's primitives of a round: requested a round ahead, the first before the counters are set up
    struct Round { u32 cnt[kPer], mask[kPer], dbits[kPer]; ushort4 r[kPer]; } next;
    auto request = [&](u32 from) {
#pragma unroll
        for (u32 j = 0; j < kPer; ++j) {
            const u32 i = from + j * kThreads + tid;
            const bool in = i - beg < share.count;
            next.cnt[j] = in ? tiles_touched[i] : 0u;
            next.r[j] = in ? rect[i] : make_ushort4(0, 0, 0, 0);
            next.mask[j] = (TIGHT && in) ? tile_masks[i] : 0u;
            next.dbits[j] = in ? __float_as_uint(depth[i]) : 0u;
        }
    };
    request(beg);
    __syncthreads();
    const u64 first = list_first_finish<kWaves>(block_offsets, beg / kPreBlock, s_part);
    for (u32 k = tid; k < entries; k += kThreads) {
        if (first + k >= list_capacity) break;
        const uint2 e = list[first + k];
        if (e.x < num_tiles) s_cur[e.x] = WIDE ? e.y : (u32)tile_offsets[e.x] + e.y;
    }
    __syncthreads();
    for (u32 from = beg; from - beg < share.count; from += kPer * kThreads) {
        const Round now = next;
        request(from + kPer * kThreads);
#pragma unroll
        for (u32 j = 0; j < kPer; ++j) {
            const u32 area = now.cnt[j] ? ((u32)now.r[j].z - (u32)now.r[j].x) * ((u32)now.r[j].w - (u32)now.r[j].y) : 0u;
            if (area == 0u || area > kMaskArea) continue;
            const u64 comp = ((u64)now.dbits[j] << 32) | (u64)(from + j * kThreads + tid);
            walk_small<TIGHT>(now.r[j], area, now.mask[j], pp.tiles_x, [&](u32 tile) {
                if (tile >= num_tiles) return;
                const u32 at = atomicAdd(&s_cur[tile], 1u);
                const u64 pos = WIDE ? tile_offsets[tile] + at : (u64)at;
                if (pos < capacity) keys[pos] = comp;
            });
        }
    }
}

// ---------------------------------------------------------------- prefix sum over the primitives
// lmk_gs_projected.offsets (optional output): exclusive prefix sum of tiles_touched -- the scan
// inside every group of 256 primitives on top of the two-level prefix sum over the groups that the
// projection stage left.  Nothing else in this stage depends on it.
__global__ __launch_bounds__(kPreBlock) void prim_offsets_kernel(
    const u32 *__restrict__ tiles_touched, u32 n, const u64 *__restrict__ block_offsets,
    const u64 *__restrict__ group_totals, u64 *__restrict__ offsets)
{
    __shared__ u64 s_gpart[kPreBlock / kWave];
    __shared__ u32 s_wave[kPreBlock / kWave];
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 i = blockIdx.x * kPreBlock + tid;
    // totals of the groups before this workgroup's own
    const u32 groups_before = blockIdx.x / kScanGroup;
    u64 part = 0;
    for (u32 g = tid; g < groups_before; g += kPreBlock) part += group_totals[g];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) part += __shfl_down(part, o, 64);
    if (lane == 0) s_gpart[wv] = part;
    const u32 cnt = i < n ? tiles_touched[i] : 0u;
    u32 incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const u32 t = __shfl_up(incl, o, 64);
        if ((int)lane >= o) incl += t;
    }
    if (lane == kWave - 1) s_wave[wv] = incl;
    __syncthreads();
    u64 base = block_offsets[blockIdx.x];
    u32 wave_base = 0, total = 0;
#pragma unroll
    for (u32 k = 0; k < kPreBlock / kWave; ++k) {
        base += s_gpart[k];
        const u32 w = s_wave[k];
        if (k < wv) wave_base += w;
        total += w;
    }
    if (i < n) offsets[i] = base + wave_base + incl - cnt;
    if (i == n - 1) offsets[n] = base + total;
}

// ---------------------------------------------------------------- per-tile sort
// On entry keys[beg .. beg + n) holds what the emit kernel wrote: depth bits << 32 | primitive index,
// the composite the list is ordered by.  On return keys/vals (or keys_out/vals_out) hold the
// sorted pairs in their final form, key = tile << 32 | depth bits, value = primitive index.
template <u32 THREADS, u32 ITEMS>
__device__ __forceinline__ void sort_pairs_in_lds(u64 *keys, u32 *vals, u64 beg, u32 n, u32 tile, u64 *s,
                                                  u64 *keys_out = nullptr, u32 *vals_out = nullptr)
{
    if (!keys_out) { keys_out = keys; vals_out = vals; }    // in place unless the caller wants the result elsewhere
    const u32 tid = team_thread<THREADS>();
    sort_in_lds<THREADS, ITEMS>(n, s, [&](u32 i) { return keys[beg + i]; });
    const u64 hi_bits = (u64)tile << 32;
    for (u32 p = tid; p < n; p += THREADS) {
        const u64 c = s[ts_slot(p)];
        keys_out[beg + p] = hi_bits | (c >> 32);
        vals_out[beg + p] = (u32)c;
    }
    team_sync<THREADS>();                                        // s may be refilled by the caller
}

// The same result for up to THREADS * ITEMS pairs with one counting step instead of the merge rounds: the
// composites go to buckets by depth, equal steps between the list's smallest and largest, as many buckets
// as pairs fit; a bucket holds one or two of them, and the place of a pair in its
// bucket is the number of smaller ones there.  Equal steps of the depth's bits instead of the depth
// (steps of equal ratio) crowd what is far into few buckets: inside a scene half of the long lists then
// fell back.
//
// What the buckets cost beyond that is the ranking, by the size of a pair's bucket on average over the pairs:
// lists of clusters of one size are even with the merge sort, less the try, at 7 (64 threads) and 22
// (512), and one large bucket holds up its wavefront.  With 1024 threads, alone on their compute unit, they are even at 56 only (200 lists of 16 384
// in clusters of 16, 22, 32, 56: all of stage 2 93, 97, 105, 122 us, by merging 123; of 8192 66, 67, 71, 81, by merging 82); the limits are
// those of 512 all the same.  Beyond these limits (a surface in front of a far background,
// equal depths) the list is left to the merge sort: returns false, nothing written.  Lists that are far beyond
// show it in a quarter of their pairs, or in their depths being one, and leave before the rest is counted.
// Called by the whole team (a workgroup, or one wavefront); cnt holds THREADS * ITEMS / 2 words, two 16-bit counters each.
//
// Bound by vector issue (half of the time of all lists together) and the latency of a list's steps; one list of 16 000 pairs
// evenly spread takes 15 us on its compute unit, in crowded buckets (15 a pair) 31, by merging 53.  So lanes talk by DPP, an atomic
// that counts also gives the pair its place in the bucket, and offsets are 32 bits wide behind a scalar base: 11.2 M -> 8.4 M
// vector instructions for the lists of up to 4096 of a 3 M overview, 35.8 -> 31.2 us; 500 000 in a cube 26.2 -> 22.6 us.
// Four pairs of a thread ranked side by side with their buckets' first three read at once: no faster.
template <u32 THREADS> struct BucketLimits {
    static constexpr u32 kMean = THREADS == 64u ? 7u : 22u;
    static constexpr u32 kMax = THREADS == 64u ? 24u : 64u;
    static constexpr u32 kProbeMax = THREADS == 64u ? 12u : 24u;     // in a quarter of the list
};

template <u32 THREADS, u32 ITEMS>
__device__ __forceinline__ bool bucket_sort_pairs(u64 *keys, u32 *vals, u64 beg, u32 n, u32 tile, u64 *s, u32 *cnt)
{
    constexpr u32 CAP = THREADS * ITEMS, kWords = ITEMS / 2, kWaves = THREADS / kWave;
    constexpr u32 kProbe = ITEMS < 4u ? 1u : ITEMS / 4u;
    using Limits = BucketLimits<THREADS>;
    static_assert(CAP < 65536u && ITEMS % 2u == 0u, "positions are 16 bits wide, two to a word");
    static_assert(CAP * Limits::kMax < (1u << 31), "the sum of the places fits a word");
    const u32 tid = team_thread<THREADS>(), lane = tid & (kWave - 1), wv = tid / kWave;
    char *const list = reinterpret_cast<char *>(keys + beg), *const indices = reinterpret_cast<char *>(vals + beg);
    u64 e[ITEMS];
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k) {                           // beyond the end its last pair again
        const u32 p = k * THREADS + tid;
        e[k] = *reinterpret_cast<const u64 *>(list + (p < n ? p : n - 1u) * 8u);
    }
#pragma unroll
    for (u32 k = 0; k < kWords; ++k) cnt[k * THREADS + tid] = 0;
    u32 lo = ~0u, hi = 0u;
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k) {
        const u32 d = (u32)(e[k] >> 32);
        lo = d < lo ? d : lo; hi = d > hi ? d : hi;
    }
    lo = wave_min(lo); hi = wave_max(hi);
    // of the wavefronts: depths, sums of the places, sums of the counts; free until the scatter
    u32 *const part = reinterpret_cast<u32 *>(s), *const places = part + 2u * kWaves, *const counts = places + kWaves, *const flag = counts + kWaves;
    if (kWaves > 1u) {
        if (tid < 2u) flag[tid] = 0u;
        if (lane == 0) { part[2 * wv] = lo; part[2 * wv + 1] = hi; }
    }
    team_sync<THREADS>();                                        // also: the counters are clear
    if (kWaves > 1u) {
#pragma unroll
        for (u32 k = 0; k < kWaves; ++k) {
            const u32 a = part[2 * k], b = part[2 * k + 1];
            lo = a < lo ? a : lo; hi = b > hi ? b : hi;
        }
    }
    // equal steps of the depth itself (positive, so its bits order alike): a pixel column holds more of what
    // is far.  A difference, a product with a positive constant and a conversion are all monotone, which is
    // all that is needed; an infinite depth is left to the merge sort.  The last counter stays free: it ends the bucket before.
    const float z0 = __uint_as_float(lo), z1 = __uint_as_float(hi);
    const float scale = z1 > z0 ? (float)CAP / (z1 - z0) : 0.0f;
    if (!(z1 < 3.0e38f) || scale == 0.0f || !(scale < 3.0e38f)) return false;         // the same for the whole team
    auto bucket = [&](u64 c) -> u32 {
        return (u32)fminf((__uint_as_float((u32)(c >> 32)) - z0) * scale, (float)(CAP - 2u));     // NaN: the last one
    };
    u32 at[ITEMS], most = 0, sum = 0;                           // at: bucket, and above it the place in the bucket, in order of arrival
    auto count = [&](u32 k) {
        at[k] = 0;
        if (k * THREADS + tid < n) {
            const u32 b = bucket(e[k]), sh = (b & 1u) * 16u;
            const u32 place = (atomicAdd(&cnt[b >> 1], 1u << sh) >> sh) & 0xffffu;
            at[k] = b | (place << 16);
            most = place > most ? place : most;
            sum += place;
        }
    };
#pragma unroll
    for (u32 k = 0; k < kProbe; ++k) count(k);
    if (team_any<THREADS>(most >= Limits::kProbeMax, flag)) return false;      // the same for the whole team
#pragma unroll
    for (u32 k = kProbe; k < ITEMS; ++k) count(k);
    bool over = most >= Limits::kMax;
    u32 total = wave_sum(sum);
    if (kWaves > 1u && lane == 0) places[wv] = total;
    if (team_any<THREADS>(over, flag + 1)) return false;        // also: every pair has been counted
    if (kWaves > 1u) {
        total = 0;
#pragma unroll
        for (u32 k = 0; k < kWaves; ++k) total += places[k];
    }
    // the sum of the squares of the counts
    if (2u * total + n > Limits::kMean * n) return false;       // the same for the whole team
    if (kWaves == 1u) team_sync<THREADS>();
    // exclusive scan: ITEMS consecutive buckets per thread
    u32 w[kWords], mine = 0;
#pragma unroll
    for (u32 k = 0; k < kWords; ++k) {
        w[k] = cnt[tid * kWords + k];
        mine += (w[k] & 0xffffu) + (w[k] >> 16);
    }
    const u32 incl = wave_scan(mine);
    u32 run = incl - mine;
    if (kWaves > 1u) {
        if (lane == kWave - 1) counts[wv] = incl;
        team_sync<THREADS>();
#pragma unroll
        for (u32 k = 0; k < kWaves; ++k) run += k < wv ? counts[k] : 0u;
    }
#pragma unroll
    for (u32 k = 0; k < kWords; ++k) {
        cnt[tid * kWords + k] = run * 0x10001u + (w[k] << 16);
        run += (w[k] & 0xffffu) + (w[k] >> 16);
    }
    team_sync<THREADS>();
    const unsigned short *const start = reinterpret_cast<const unsigned short *>(cnt);
#pragma unroll
    for (u32 k = 0; k < ITEMS; ++k)
        if (k * THREADS + tid < n) s[start[at[k] & 0xffffu] + (at[k] >> 16)] = e[k];
    team_sync<THREADS>();
    const u64 hi_bits = (u64)tile << 32;
#pragma unroll 2
    for (u32 p = tid; p < n; p += THREADS) {
        const u64 c = s[p];
        const u32 b = bucket(c), end = start[b + 1u];
        u32 to = start[b];
        for (u32 j = to; j < end; ++j) to += s[j] < c ? 1u : 0u;
        *reinterpret_cast<u64 *>(list + to * 8u) = hi_bits | (c >> 32);
        *reinterpret_cast<u32 *>(indices + to * 4u) = (u32)c;
    }
    return true;
}

// a list of 1 .. THREADS * ITEMS pairs, in place; s: list_words(THREADS * ITEMS) words.  The counters lie behind
// the composites, where the merge sort has the end of its padded ones: 40 KB for 4096 pairs, so that four
// workgroups fit a compute unit; 160 KB, all that there is, for 16384.
constexpr u32 list_words(u32 pairs) { return pairs + pairs / 4u; }
template <u32 THREADS, u32 ITEMS>
__device__ __forceinline__ void sort_list(u64 *keys, u32 *vals, u64 beg, u32 n, u32 tile, u64 *s)
{
    constexpr u32 CAP = THREADS * ITEMS;
    static_assert(CAP + CAP / 16u <= list_words(CAP), "the merge sort fits as well");
    if (bucket_sort_pairs<THREADS, ITEMS>(keys, vals, beg, n, tile, s, reinterpret_cast<u32 *>(s + CAP))) return;
    team_sync<THREADS>();                                        // `s` is free again
    sort_pairs_in_lds<THREADS, ITEMS>(keys, vals, beg, n, tile, s);
}

// ---------------------------------------------------------------- lists beyond kHuge pairs
__device__ __forceinline__ bool pair_less(u64 ka, u32 va, u64 kb, u32 vb)
{
    return ka < kb || (ka == kb && va < vb);
}

// Merge-path split by one wavefront: the number of elements of A = [a0, a1) among the first
// `diag` outputs of the merge of A and B = [a1, b1) (sorted runs in global memory).  Every
// round the 64 lanes probe 64 evenly spaced candidates, which narrows the range 64-fold.
__device__ __forceinline__ u64 wave_merge_split(const u64 *__restrict__ sk, const u32 *__restrict__ sv,
                                                u64 a0, u64 a1, u64 b1, u64 diag, u32 lane)
{
    const u64 lenA = a1 - a0, lenB = b1 - a1;
    u64 lo = diag > lenB ? diag - lenB : 0, hi = diag < lenA ? diag : lenA;
    while (lo < hi) {                                       // wave-uniform
        const u64 step = (hi - lo + 63) / 64;
        const u64 m = lo + (u64)(lane + 1) * step - 1;
        bool p = false;
        if (m < hi) {
            const u64 jb = a1 + (diag - 1 - m);
            p = pair_less(sk[a0 + m], sv[a0 + m], sk[jb], sv[jb]);
        }
        const u64 c = (u64)__builtin_popcountll(__builtin_amdgcn_ballot_w64(p));   // leading run of "true"
        const u64 nlo = lo + c * step;
        const u64 nhi = lo + (c + 1) * step - 1;
        hi = nhi < hi ? nhi : hi;
        lo = nlo;
    }
    return lo;
}

// A list of L > kHuge pairs by a workgroup of 1024 threads: chunks of kHuge pairs are sorted in LDS, then merged
// pairwise (run length doubling) between the two pair buffers, kHuge outputs at a time: sixteen wavefronts find the
// splits of sixteen output segments, then each segment's two input windows are staged in
// LDS, merged there and written out coalesced.  The result ends in keys/vals.  s: kHuge + kHuge / 16 composites and
// behind them two words per wavefront.
__device__ __forceinline__ void sort_huge_list(u64 *__restrict__ keys, u32 *__restrict__ vals, u64 *__restrict__ keys_alt,
                                               u32 *__restrict__ vals_alt, u64 beg, u64 L, u32 tile, u64 *s)
{
    u64 *s_split = s + kHuge + kHuge / 16;
    const u32 tid = team_thread<kHugeThreads>(), lane = tid & (kWave - 1), wv = tid / kWave;
    constexpr u32 kWaves = kHugeThreads / kWave;

    // an odd number of merge rounds: the chunk sorts write to the alternate buffers, so that the
    // last round ends in keys/vals either way
    u32 rounds = 0;
    for (u64 run = kHuge; run < L; run <<= 1) ++rounds;
    const bool start_alt = (rounds & 1u) != 0u;
    u64 *k0 = start_alt ? keys_alt : keys, *k1 = start_alt ? keys : keys_alt;
    u32 *v0 = start_alt ? vals_alt : vals, *v1 = start_alt ? vals : vals_alt;
    for (u64 c0 = 0; c0 < L; c0 += kHuge) {
        const u32 n = (u32)(L - c0 < (u64)kHuge ? L - c0 : (u64)kHuge);
        if (n >= 2) sort_pairs_in_lds<kHugeThreads, kHugeItems>(keys, vals, beg + c0, n, tile, s, k0, v0);
        else if (tid == 0) {                                 // a chunk of one pair: only its form changes
            const u64 c = keys[beg + c0];
            k0[beg + c0] = ((u64)tile << 32) | (c >> 32); v0[beg + c0] = (u32)c;
        }
    }
    // the chunk sorts of this workgroup wrote the runs the merges read
    __threadfence_block();
    __syncthreads();

    u64 *sk = k0 + beg, *dk = k1 + beg;
    u32 *sv = v0 + beg, *dv = v1 + beg;
    const u64 hi_bits = (u64)tile << 32;
    const u64 nseg = (L + kHuge - 1) / kHuge;
    for (u64 run = kHuge; run < L; run <<= 1) {
        for (u64 seg0 = 0; seg0 < nseg; seg0 += kWaves) {
            {   // wavefront wv: the splits at both ends of output segment seg0 + wv
                const u64 seg = seg0 + wv;
                if (seg < nseg) {
                    const u64 o = seg * kHuge;
                    const u64 a0 = (o / (2 * run)) * (2 * run);
                    const u64 a1 = a0 + run < L ? a0 + run : L;
                    const u64 b1 = a0 + 2 * run < L ? a0 + 2 * run : L;
                    const u64 oe = o + kHuge < b1 ? o + kHuge : b1;
                    const u64 i0 = wave_merge_split(sk, sv, a0, a1, b1, o - a0, lane);
                    const u64 i1 = wave_merge_split(sk, sv, a0, a1, b1, oe - a0, lane);
                    if (lane == 0) { s_split[2 * wv] = i0; s_split[2 * wv + 1] = i1; }
                }
            }
            __syncthreads();
            for (u32 w = 0; w < kWaves && seg0 + w < nseg; ++w) {
                const u64 o = (seg0 + w) * kHuge;
                const u64 a0 = (o / (2 * run)) * (2 * run);
                const u64 a1 = a0 + run < L ? a0 + run : L;
                const u64 b1 = a0 + 2 * run < L ? a0 + 2 * run : L;
                const u64 oe = o + kHuge < b1 ? o + kHuge : b1;
                const u64 i0 = s_split[2 * w], i1 = s_split[2 * w + 1];
                const u64 j0 = (o - a0) - i0;                // elements of B before the segment
                const u32 la = (u32)(i1 - i0), total = (u32)(oe - o);
                // stage A[i0, i1) then B[j0, j0 + total - la) as composites
                for (u32 p = tid; p < total; p += kHugeThreads) {
                    const u64 src = p < la ? a0 + i0 + p : a1 + j0 + (p - la);
                    s[ts_slot(p)] = (sk[src] << 32) | (u64)sv[src];
                }
                __syncthreads();
                const u32 o0 = tid * kHugeItems;
                u64 e[kHugeItems];
                if (o0 < total) merge_from_lds<kHugeItems>(s, 0u, la, total, o0, e);
                __syncthreads();
                if (o0 < total) {
#pragma unroll
                    for (u32 k = 0; k < kHugeItems; ++k)
                        if (o0 + k < total) s[ts_slot(o0 + k)] = e[k];
                }
                __syncthreads();
                for (u32 p = tid; p < total; p += kHugeThreads) {
                    const u64 c = s[ts_slot(p)];
                    dk[o + p] = hi_bits | (c >> 32);
                    dv[o + p] = (u32)c;
                }
                __syncthreads();
            }
        }
        // this workgroup's writes of the round are read by all its threads in the next one
        __threadfence_block();
        __syncthreads();
        u64 *tk = sk; sk = dk; dk = tk;
        u32 *tv = sv; sv = dv; dv = tv;
    }
}

// ---------------------------------------------------------------- the launches of the per-tile sort
// The lists beyond kMid pairs, the first of `order`: one workgroup each, up to kHuge pairs whole in the LDS of a compute unit.
// Such a list was cut into chunks of 4096 before, sorted with the lists of up to 4096 and merged in two rounds, which took
// two launches more (four in all; 3 M overview, 85 long lists 75 -> 62 us, 20 M of a city 88 -> 60, and where no list is long
// the launches themselves: 1.2 M inside 20 -> 12, 30 011 at 333 x 217 22 -> 10).  No more workgroups than compute units: an idle
// one would wait for all of one's LDS.
__global__ __launch_bounds__(kHugeThreads) void tile_sort_long_kernel(
    u64 *__restrict__ keys, u32 *__restrict__ vals, u64 *__restrict__ keys_alt, u32 *__restrict__ vals_alt,
    const u64 *__restrict__ tile_offsets, const u32 *__restrict__ order, const u32 *__restrict__ classes, u32 num_tiles)
{
    __shared__ __attribute__((aligned(16))) u64 s[list_words(kHuge)];
    static_assert(kHuge + kHuge / 16 + 2 * (kHugeThreads / kWave) <= list_words(kHuge), "the merges fit as well");
    u32 lists = classes[0] + classes[3];
    const u32 elsewhere = classes[kDenseClass];
    if (elsewhere) return;
    if (lists > num_tiles) lists = num_tiles;               // cannot happen with a consistent table
    for (u32 k = blockIdx.x; k < lists; k += gridDim.x) {
        const u32 tile = order[k];
        if (tile >= num_tiles) continue;
        const u64 beg = tile_offsets[tile];
        const u64 len = tile_offsets[tile + 1] - beg;
        if (len > (u64)kHuge) sort_huge_list(keys, vals, keys_alt, vals_alt, beg, len, tile, s);
        else if (len > (u64)kHuge / 2) sort_list<kHugeThreads, kHugeItems>(keys, vals, beg, (u32)len, tile, s);
        else if (len > 1) sort_list<kHugeThreads, kHugeItems / 2>(keys, vals, beg, (u32)len, tile, s);
        __syncthreads();                                    // `s` is free again
    }
}

// Lists of up to kMid pairs: one workgroup each above kSmallCap pairs, one wavefront each below.  (Two pairs a thread for up to 1024
// takes as long as four.)
constexpr u32 kShortPerBlock = kMidThreads / kSmallThreads;
__global__ __launch_bounds__(kMidThreads, 8) void tile_sort_kernel(
    u64 *__restrict__ keys, u32 *__restrict__ vals, const u64 *__restrict__ tile_offsets,
    const u32 *__restrict__ order, const u32 *__restrict__ classes, u32 num_tiles,
    ScratchHeader *__restrict__ header, u32 *__restrict__ tile_count)
{
    constexpr u32 kShortWords = list_words(kSmallCap);      // LDS of a wavefront's own list
    static_assert(kShortPerBlock * kShortWords <= list_words(kMid), "a share each");
    __shared__ __attribute__((aligned(16))) u64 s[list_words(kMid)];
    const u32 first = classes[0] + classes[3], mid = classes[1], low = classes[2], elsewhere = classes[kDenseClass];
    // the scan has read the per-tile counters (both halves) and the emit kernel has consumed the
    // deferred list: leave them empty for the next call
    const u32 tid = threadIdx.x;
    for (u32 t = blockIdx.x * kMidThreads + tid; t < 2u * (num_tiles + 1u); t += gridDim.x * kMidThreads) tile_count[t] = 0;
    if (blockIdx.x == 0 && tid == 0) { header->big_count = 0; header->giant_count = 0; }
    const u32 whole = mid + low;
    if (elsewhere || (u64)first + whole > num_tiles) return;    // the second cannot happen with a consistent table
    const u32 wv = (u32)__builtin_amdgcn_readfirstlane((int)(tid / kWave)), b = blockIdx.x;     // the same for the wavefront
    const u32 k = b < whole ? first + b : first + whole + (b - whole) * kShortPerBlock + wv;
    if (k >= num_tiles) return;
    const u32 tile = order[k];
    if (tile >= num_tiles) return;
    const u64 beg = tile_offsets[tile];
    const u64 len = tile_offsets[tile + 1] - beg;
    if (b < whole) {                                        // the same for the workgroup
        if (len < 2 || len > (u64)kMid) return;             // cannot happen with a consistent table
        if (len > (u64)kLow) sort_list<kMidThreads, 8u>(keys, vals, beg, (u32)len, tile, s);
        else sort_list<kMidThreads, 4u>(keys, vals, beg, (u32)len, tile, s);
        return;
    }
    // from here on every wavefront goes its own way
    if (len < 1 || len > (u64)kSmallCap) return;
    if (len == 1) {                                         // nothing to sort: only the pair's form changes
        if ((tid & (kWave - 1u)) == 0u) {
            const u64 c = keys[beg];
            keys[beg] = ((u64)tile << 32) | (c >> 32); vals[beg] = (u32)c;
        }
        return;
    }
    u64 *my_s = s + wv * kShortWords;
    // fewer elements per lane for shorter lists
    if (len <= 2u * kSmallThreads) sort_list<kSmallThreads, 2u>(keys, vals, beg, (u32)len, tile, my_s);
    else if (len <= 4u * kSmallThreads) sort_list<kSmallThreads, 4u>(keys, vals, beg, (u32)len, tile, my_s);
    else sort_list<kSmallThreads, kSmallItems>(keys, vals, beg, (u32)len, tile, my_s);
}

// The other way's lists.  As part of the sort launch it would take registers from the lists of all frames whose buffers could hold such a
// frame; a launch that leaves at once costs these frames 2 us.
template <bool TIGHT, bool RECORDS>
__global__ __launch_bounds__(kDenseThreads, 5) void dense_emit_kernel(
    u64 *__restrict__ keys, u32 *__restrict__ vals, const u64 *__restrict__ tile_offsets, u64 capacity,
    const ScratchHeader *__restrict__ header, const u32 *__restrict__ classes, DenseArgs dense)
{
    __shared__ __attribute__((aligned(16))) u64 s[kDenseWaves * (u32)((RECORDS ? sizeof(EmitRuns) : sizeof(EmitSpace)) / sizeof(u64))];
    if (!classes[kDenseClass]) return;
    dense_emit<TIGHT, RECORDS>(dense, header, tile_offsets, capacity, keys, vals, s);
}

// ---------------------------------------------------------------- launcher
hipError_t launch_bin_sort(const lmk_gs_projected &proj, u32 n, const ProjParams &pp, const lmk_gs_binned &out,
                           char *scratch, const ScratchLayout &L, hipStream_t stream)
{
    ScratchHeader *header = reinterpret_cast<ScratchHeader *>(scratch + L.header);
    const u32 num_tiles = pp.tiles_x * pp.tiles_y;
    u32 *tile_count = reinterpret_cast<u32 *>(scratch + L.tile_count);
    u32 *large_count = tile_count + (num_tiles + 1);
    const u64 *block_offsets = reinterpret_cast<const u64 *>(scratch + L.block_offsets);
    const u64 *group_totals = reinterpret_cast<const u64 *>(scratch + L.group_totals);
    const u32 *tile_masks = reinterpret_cast<const u32 *>(scratch + L.tile_masks);
    u32 *bin_count = reinterpret_cast<u32 *>(scratch + L.bin_count);
    u32 *tile_cursor = reinterpret_cast<u32 *>(scratch + L.tile_cursor);
    u32 *big_idx = reinterpret_cast<u32 *>(scratch + L.big_idx);
    u32 *order = reinterpret_cast<u32 *>(scratch + L.order);
    u32 *classes = reinterpret_cast<u32 *>(scratch + L.classes);
    const ushort4 *rect = reinterpret_cast<const ushort4 *>(proj.rect);
    const float4 *feat = reinterpret_cast<const float4 *>(proj.feat);
    // the (tile, start) lists of the counting workgroups live in the alternate key buffer, which
    // nothing else uses before the merge rounds of the per-tile sort; a list has at most one entry
    // per pair of its workgroup and starts at the number of pairs before the workgroup
    uint2 *list = reinterpret_cast<uint2 *>(out.keys_alt);
    const bool tight = pp.cam.binning == 1u;
    const bool wide = out.capacity > 0xffffffffull;
    const u32 lds_tiles = num_tiles <= kLdsTilesSmall ? kLdsTilesSmall : (num_tiles <= kLdsTilesLarge ? kLdsTilesLarge : 0u);
    const u32 bin_threads = lds_tiles == kLdsTilesSmall ? BinShape<kLdsTilesSmall>::kThreads : BinShape<kLdsTilesLarge>::kThreads;
    // the listed primitives are walked by fixed grids striding over the two lists: as workgroups of
    // kLargeThreads threads in the counting pass, as workgroups of the emit kernel behind its own
    const u32 large_blocks = 4u * L.bin_blocks < kLargeBlocks ? 4u * L.bin_blocks : kLargeBlocks;
    const u32 giant_blocks = L.bin_blocks < kGiantBlocks ? L.bin_blocks : kGiantBlocks;
    const u32 large_blocks_emit = (large_blocks * kLargeThreads + bin_threads - 1) / bin_threads;
    hipError_t e;

    // the launches that both ways share: `with` is called with what their kernels get of the other one
    const u64 dense_min = dense_min_pairs(n, out, pp.tiles_x, pp.tiles_y);
    const bool dense = dense_min != ~0ull;
    const DenseLayout DL = dense_layout(n, out.capacity, pp.tiles_x, pp.tiles_y);
    const u32 dense_grid = dense ? dense_blocks(DL) : 0u;
    auto both = [&](auto with) {
        if (dense) with(dense_args(proj, n, pp, out, DL, dense_min)); else with(OneWay());
    };
    auto most = [](u32 a, u32 b) { return a > b ? a : b; };
    if (L.bin_blocks > 0) {
        both([&](auto d) {
            using Dense = decltype(d);
            auto count = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(Dense::kDense ? most(L.bin_blocks, DL.chunks) : L.bin_blocks), dim3(bin_threads), 0, stream,
                                   proj.tiles_touched, rect, tile_masks, n, pp.tiles_x, num_tiles, tile_count, header, big_idx,
                                   reinterpret_cast<const u32 *>(scratch + L.block_sums), L.pre_blocks,
                                   block_offsets, group_totals, bin_count, list, out.capacity, d);
            };
            if (lds_tiles == kLdsTilesSmall) { if (tight) count(count_kernel<kLdsTilesSmall, true, Dense>); else count(count_kernel<kLdsTilesSmall, false, Dense>); }
            else if (lds_tiles == kLdsTilesLarge) { if (tight) count(count_kernel<kLdsTilesLarge, true, Dense>); else count(count_kernel<kLdsTilesLarge, false, Dense>); }
            else { if (tight) count(count_kernel<0u, true, Dense>); else count(count_kernel<0u, false, Dense>); }
            if constexpr (Dense::kDense) launch_depth_rank(out, DL, d, header, stream);
            auto count_large = [&](auto kernel) {
                const u32 blocks = giant_blocks + large_blocks;
                hipLaunchKernelGGL(kernel, dim3(most(blocks, dense_grid)), dim3(kLargeThreads), 0, stream,
                                   rect, feat, pp, n, num_tiles, large_count, header, big_idx, giant_blocks, blocks, tile_count, d);
            };
            if (tight) count_large(count_large_kernel<true, Dense>); else count_large(count_large_kernel<false, Dense>);
        });
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    auto scan = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(2), dim3(kScanThreads), 0, stream,
                           tile_count, large_count, num_tiles, out.capacity, header, out.tile_offsets, tile_cursor,
                           n == 0 ? proj.offsets : nullptr, order, out.tile_order, classes, dense_min);
    };
    if (num_tiles <= kLdsTilesSmall) scan(tile_scan_kernel<1u>);
    else if (num_tiles <= kLdsTilesLarge) scan(tile_scan_kernel<4u>);
    else scan(tile_scan_kernel<0u>);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (L.bin_blocks > 0) {
        auto emit = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(L.bin_blocks + giant_blocks + large_blocks_emit), dim3(bin_threads), 0, stream,
                               proj.tiles_touched, rect, proj.depth, feat, tile_masks, n, pp, num_tiles,
                               out.tile_offsets, tile_cursor, header, big_idx, block_offsets, group_totals,
                               bin_count, list, out.capacity, L.bin_blocks, giant_blocks, out.capacity, out.keys, classes);
        };
        auto emit_for = [&](auto lds_tag) {
            constexpr u32 LT = decltype(lds_tag)::value;
            if (tight) { if (wide) emit(emit_kernel<LT, true, true>); else emit(emit_kernel<LT, true, false>); }
            else { if (wide) emit(emit_kernel<LT, false, true>); else emit(emit_kernel<LT, false, false>); }
        };
        if (lds_tiles == kLdsTilesSmall) emit_for(std::integral_constant<u32, kLdsTilesSmall>());
        else if (lds_tiles == kLdsTilesLarge) emit_for(std::integral_constant<u32, kLdsTilesLarge>());
        else emit_for(std::integral_constant<u32, 0u>());
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (proj.offsets) {
            hipLaunchKernelGGL(prim_offsets_kernel, dim3(L.pre_blocks), dim3(kPreBlock), 0, stream,
                               proj.tiles_touched, n, block_offsets, group_totals, proj.offsets);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    // The long lists first, a workgroup a compute unit at most (each takes all of its LDS); none if the buffers do not hold that
    // many pairs.  The others' grid is an upper bound from the capacity, surplus workgroups leave at once.
    auto at_most = [](u64 a, u64 b) { return (u32)(a < b ? a : b); };
    if (out.capacity > kMid)
        hipLaunchKernelGGL(tile_sort_long_kernel, dim3(at_most(at_most(out.capacity / (kMid + 1u), num_tiles), kLongBlocks)), dim3(kHugeThreads), 0, stream,
                           out.keys, out.vals, out.keys_alt, out.vals_alt, out.tile_offsets, order, classes, num_tiles);
    const u32 whole = at_most(out.capacity / (kSmallCap + 1u), num_tiles), shorts = (num_tiles + kShortPerBlock - 1) / kShortPerBlock;
    hipLaunchKernelGGL(tile_sort_kernel, dim3(whole + shorts), dim3(kMidThreads), 0, stream,
                       out.keys, out.vals, out.tile_offsets, order, classes, num_tiles, header, tile_count);
    if (dense) {
        const DenseArgs d = dense_args(proj, n, pp, out, DL, dense_min);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(dense_grid), dim3(kDenseThreads), 0, stream,
                               out.keys, out.vals, out.tile_offsets, out.capacity, header, classes, d);
        };
        if (d.records) { if (tight) go(dense_emit_kernel<true, true>); else go(dense_emit_kernel<false, true>); }
        else if (tight) go(dense_emit_kernel<true, false>);
        else go(dense_emit_kernel<false, false>);
    }
    return hipGetLastError();
}

}  // namespace lmk
