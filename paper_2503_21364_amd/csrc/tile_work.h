// Which tiles, and whether whole or shared, the workgroups of the compositing kernel and of its gradient take.
//
// A tile's workgroup takes its list from front to back.  An image of a few hundred tiles then leaves most of the chip idle, and
// one with a few very long lists waits for these.  Such tiles are shared by four workgroups: of the compositing each takes an
// 8x8 block, a wavefront per 4x4 cell, four lanes a pixel with an entry each; of the gradient a part of the list.  Either way
// takes about twice the vector instructions, so that it is the better one only where the image would wait:
//  * images of up to kSharedTiles tiles: all tiles;
//  * of up to kSharedMaxTiles, with the caller's order by list length: those whose list has a 1 / kSharedPairs of the
//    frame's pairs (no more than kSharedPairs tiles have, and they are the first of the order);
//  * else none (a 3 M overview at 1080p has no such list among 8160).
// Every workgroup looks at a few places of the order to see how many first places hold all the long lists, rounded up; four
// workgroups of each of these come first, then the other places, then idle ones for the shares that this image does not have.
// The shares of a tile are on one die, so that they read the same records through one L2, and on different compute units of it.
// What the looks cost, and the idle workgroups, is 1 us where no list is long.
//
// Measured, us, compositing, every tile whole / so: 30 011 primitives at 640 x 480 28.6 / 29.7, at 333 x 217 43 / 25; 1 M in clusters at
// 400 x 300 236 / 160; 3 M of a city at 400 x 300 130 / 67; 10 000 at 256 x 256, a frame, all shares of a tile on one compute
// unit 73.0, so 65.7.
#ifndef LMK_GS_TILE_WORK_H
#define LMK_GS_TILE_WORK_H
#include "lmk_gs_internal.h"

namespace lmk {

constexpr u32 kSharedTiles = 256, kSharedMaxTiles = 2048, kSharedPairs = 256;
static_assert(kSharedPairs <= kSharedTiles, "every image with an order has as many places");

// the shortest list that has a 1 / kSharedPairs of them
__host__ __device__ __forceinline__ u64 long_list_from(u64 pairs) { return (pairs + (kSharedPairs - 1u)) / kSharedPairs; }

// Which of `apart` places, a multiple of eight, workgroup `b` of share `share` of them takes.  Workgroups go to the dies in turn, and on
// a die to its 32 compute units: a quarter of the places further with each share, so that the shares of a tile are on four
// of these.
__host__ __device__ __forceinline__ u32 shared_place(u32 b, u32 share, u32 apart)
{
    const u32 groups = apart >> 3, turned = (b >> 3) + groups - share * ((groups + 3u) >> 2) % groups;
    return (turned < groups ? turned : turned - groups) * 8u + (b & 7u);
}

// number of workgroups
__host__ __device__ __forceinline__ u32 tile_work_grid(u32 num_tiles, bool ordered)
{
    if (num_tiles <= kSharedTiles) return 4u * ((num_tiles + 7u) & ~7u);
    return ordered && num_tiles <= kSharedMaxTiles ? num_tiles + 3u * kSharedPairs : num_tiles;
}

// what workgroup `b` of them takes: a whole tile, or a share of one; num_tiles: none.  In images of more than kSharedTiles tiles none is
// shared if more than `most` lists are long.
struct TileWork { u32 whole, shared, share; };
__device__ __forceinline__ TileWork tile_work(u32 b, u32 num_tiles, const u32 *__restrict__ tile_order,
                                              const u64 *__restrict__ tile_offsets, u32 most = kSharedPairs)
{
    auto at = [&](u32 place) {                                          // num_tiles for a corrupt hint too
        const u32 t = place < num_tiles ? (tile_order ? tile_order[place] : place) : num_tiles;
        return t < num_tiles ? t : num_tiles;
    };
    if (num_tiles <= kSharedTiles) {
        const u32 apart = (num_tiles + 7u) & ~7u, share = b / apart;
        return { num_tiles, at(shared_place(b - share * apart, share, apart)), share };
    }
    if (!tile_order || num_tiles > kSharedMaxTiles) return { at(b), num_tiles, 0u };
    const u64 min_long = long_list_from(tile_offsets[num_tiles]);
    auto is_long = [&](u32 t) { return tile_offsets[t + 1] - tile_offsets[t] >= min_long; };
    // two trips to memory for all of them: without the barrier the compiler waits for each length by itself
    constexpr u32 kLooks = 6, look[kLooks + 1] = { 0u, 16u, 32u, 64u, 128u, 192u, 256u };
    static_assert(look[kLooks] == kSharedPairs, "room for all long lists, and the grid has a workgroup for each of their shares");
    u64 from[kLooks], to[kLooks];
#pragma unroll
    for (u32 k = 0; k < kLooks; ++k) {
        u32 t = tile_order[look[k]];
        t = t < num_tiles ? t : num_tiles - 1u;
        from[k] = tile_offsets[t]; to[k] = tile_offsets[t + 1];
    }
    __builtin_amdgcn_sched_barrier(0);
    u32 places = 0;
#pragma unroll
    for (u32 k = 0; k < kLooks; ++k) places = to[k] - from[k] >= min_long ? look[k + 1] : places;
    if (places > most) places = 0u;
    if (b >= 4u * places) return { at(b - 3u * places), num_tiles, 0u };
    const u32 share = b / places, t = at(shared_place(b - share * places, share, places));
    if (t < num_tiles && is_long(t)) return { num_tiles, t, share };
    return { share == 0u ? t : num_tiles, num_tiles, 0u };
}

}  // namespace lmk
#endif
