// Which tiles, and whether whole or shared, the workgroups of the compositing kernel and of its gradient take.
//
// A tile's workgroup takes its list from front to back.  An image of a few hundred tiles then leaves most of the chip idle, and
// one with a few very long lists waits for these.  Such tiles are shared by four workgroups: of the compositing each takes an
// 8x8 block, a wavefront per 4x4 cell, four lanes a pixel with an entry each; of the gradient a part of the list.  Either way
// takes about twice the vector instructions, so that it is the better one only where the image would wait:
//  * images of up to kSharedTiles tiles: all tiles;
//  * of up to kSharedMaxTiles, with the caller's order by list length: those of the first kSharedPlaces places whose list
//    has a 1 / kSharedPairs of the frame's pairs, if there is room for three helpers each (below);
//  * else none (a 3 M overview at 1080p has no such list among 8160).
// The helpers are the workgroups of the shortest lists, which take their share when their own tile is done, and idle ones that
// make up the number in images of fewer tiles; a place has helpers always in images of up to kSharedHelpers tiles.  Workgroups for
// every share that there might be cost 2 to 5 us where these are not; working out beforehand, in every workgroup, how many
// tiles are shared cost 3 (30 000 primitives at 640 x 480: 27.8 us unshared, 31.6 so, 28.1 with the helpers).  Helpers have to be
// short of work: if the longest helper's list has a 1 / (4 kSharedPairs) of the pairs or less all places are served; else only those
// with idle helpers are, and only where the list is twice as long as the first that goes without, as the image would wait
// for that one all the same (200 000 evenly in a cube, 414 tiles, training step: 297 us without this line, 279 with it or unshared).
// A tile's workgroups decide from a few places of the order, all alike; which they are is the same for all.  The shares of a tile are a
// multiple of the eight dies apart, so that they read the same records through one L2.
//
// Measured, us, compositing and its gradient, every tile whole / so: 30 000 primitives at 333 x 217 43, 140 / 27, 96; 1 M in
// clusters, 400 x 300, 291, 1184 / 148, 685, 800 x 600 176, 663 / 122, 463; 200 000 evenly in a cube, 256 x 256, 57, 199 / 49, 144, 400 x 300
// 49, 165 / 46, 149, 800 x 600 38, 142 / 36, 133 (of these last the lists are not shared: other steps).
#ifndef LMK_GS_TILE_WORK_H
#define LMK_GS_TILE_WORK_H
#include "lmk_gs_internal.h"

namespace lmk {

constexpr u32 kSharedTiles = 256, kSharedMaxTiles = 2048, kSharedPairs = 256, kSharedPlaces = 128;
constexpr u32 kSharedHelpers = 3u * kSharedPlaces;
static_assert(kSharedPlaces % 8u == 0u && 2u * kSharedPlaces <= kSharedTiles, "the places lie in the longer half of the order");

__host__ __device__ __forceinline__ u32 order_half(u32 num_tiles) { return ((num_tiles + 15u) >> 4) * 8u; }
__host__ __device__ __forceinline__ u32 idle_helpers(u32 num_tiles)
{
    const u32 half = order_half(num_tiles);
    if (num_tiles <= kSharedHelpers) return kSharedHelpers;
    return half < kSharedHelpers ? kSharedHelpers - half : 0u;
}

// number of workgroups
__host__ __device__ __forceinline__ u32 tile_work_grid(u32 num_tiles, bool ordered)
{
    if (num_tiles <= kSharedTiles) return 4u * ((num_tiles + 7u) & ~7u);
    return ordered && num_tiles <= kSharedMaxTiles ? 2u * order_half(num_tiles) + idle_helpers(num_tiles) : num_tiles;
}

// what workgroup `b` of them takes: a whole tile, then one of the four shares of another; num_tiles: none
struct TileWork { u32 whole, shared, share; };
__host__ __device__ __forceinline__ TileWork tile_work(u32 b, u32 num_tiles, const u32 *__restrict__ tile_order,
                                                       const u64 *__restrict__ tile_offsets)
{
    auto at = [&](u32 place) {                                          // num_tiles for a corrupt hint too
        const u32 t = place < num_tiles ? (tile_order ? tile_order[place] : place) : num_tiles;
        return t < num_tiles ? t : num_tiles;
    };
    if (num_tiles <= kSharedTiles) {
        const u32 apart = (num_tiles + 7u) & ~7u, share = b / apart;
        return { num_tiles, at(b - share * apart), share };
    }
    if (!tile_order || num_tiles > kSharedMaxTiles) return { at(b), num_tiles, 0u };
    // workgroups: the longer half of the places, the idle helpers, the shorter half.  Helpers: the idle ones, then from the
    // last place on (by eights, in their order)
    const u32 half = order_half(num_tiles), idle = idle_helpers(num_tiles);
    auto from_end = [&](u32 i) { return half - 8u - (i & ~7u) + (i & 7u); };
    auto length = [&](u32 t) { return t < num_tiles ? tile_offsets[t + 1] - tile_offsets[t] : 0ull; };
    const bool longer = b < half, own = longer || b >= half + idle;
    const u32 place = longer ? b : b - idle;
    const u32 helper = longer ? kSharedHelpers : (own ? idle + from_end(b - half - idle) : b - half);
    const u32 of = longer ? place : (helper < kSharedHelpers ? helper / 24u * 8u + (helper & 7u) : kSharedPlaces);
    u32 shared = num_tiles;
    if (of < kSharedPlaces) {
        const u32 served = idle / 24u * 8u;                             // places with idle helpers
        const u32 t = at(of), next = at(served);
        const u32 longest = idle < kSharedHelpers ? at(half + from_end(kSharedHelpers - 1u - idle)) : num_tiles;
        const u64 len = length(t), pairs = tile_offsets[num_tiles];
        const bool room = length(longest) * (4u * kSharedPairs) <= pairs || (of < served && len >= 2u * length(next));
        if (len * kSharedPairs >= pairs && room) shared = t;
    }
    return { own && !(longer && shared < num_tiles) ? at(place) : num_tiles, shared, longer ? 0u : 1u + (helper >> 3) % 3u };
}

}  // namespace lmk
#endif
