// Internal declarations shared by the translation units of liblmk_gs.so.
// Not part of the public ABI (include/lmk_gs.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lmk_gs.h"

namespace lmk {

typedef uint64_t u64;
typedef uint32_t u32;

constexpr u32 kWave = 64;               // CDNA wavefront width
constexpr u32 kPreBlock = LMK_GS_PRE_BLOCK;   // primitives per preprocess workgroup
constexpr u32 kScanGroup = 256;         // preprocess workgroups per group of the two-level prefix sum
// The counting and emit kernels keep one counter per tile in LDS: up to 8192 tiles (1080p has
// 8160) in 32 KB, up to 32768 (2160p has 32400) in 128 KB.  Larger images take the route of the
// large rectangles for every primitive: one global atomic per pair.
constexpr u32 kLdsTilesSmall = 8192, kLdsTilesLarge = 32768;

// LDS accesses of one wavefront complete in program order: only the compiler has to keep to it
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Header at the start of the scratch buffer.
struct ScratchHeader {
    u64 dup_count;      // D = pairs of the frame = sum of tiles_touched (known when lmk_gs_preprocess is done)
    int32_t status;     // LMK_GS_* code of the frame's latest stage 2 (LMK_GS_OK after stage 1)
    u32 ordered;        // the projection had an index: the primitives are in its order
    u32 big_count;      // stage 2: primitives on the deferred list, from the front (one wavefront each)
    u32 giant_count;    // ... and from the back (one workgroup each)
    u64 counted;        // dup_count as the counting kernels saw it: the scan puts the sum of the lists in its place
    u64 looks;          // without an index: pairs of primitives looked at, and above them how many of them lie near one another
};

// Carving of the caller's scratch buffer (all offsets multiples of 256 bytes).  The part up to
// `bin_count` is what lmk_gs_preprocess touches; it depends on n and the image size only.
struct ScratchLayout {
    size_t header;        // ScratchHeader
    size_t tile_count;    // u32 [2][tiles + 1]  pairs per tile in the counting workgroups' runs / of the listed primitives:
                          //                     zero between frames, accumulated by the counting kernels
    size_t block_sums;    // u32 [pre_blocks]      tile counts per preprocess workgroup (256 primitives)
    size_t block_offsets; // u64 [pre_blocks + 1]  their exclusive prefix sum within groups of kScanGroup
    size_t group_totals;  // u64 [groups]          total of each group
    size_t tile_masks;    // u32 [n]           binning rule 1: kept tiles of rectangles of up to 32 tiles
    size_t bin_count;     // u32 [bin_blocks]  entries in each counting workgroup's list of (tile, start of its run)
    size_t tile_cursor;   // u32 [tiles + 1] running position of the listed primitives' pairs inside every tile's slice
    size_t big_idx;       // u32 [n]         deferred list: primitives whose rectangles are walked by wavefronts of their own
    size_t order;         // u32 [tiles]     tile ids by descending list length
    size_t classes;       // u32 [8]         tiles per size class of the per-tile sort (see tile_scan_kernel)
    size_t spare;         // 8 bytes [capacity / 2048 + 2]  no kernel's; the workspace keeps the size that callers have planned with
    size_t total;
    u32 pre_blocks;       // ceil(n / kPreBlock)
    u32 bin_blocks;       // counting workgroups: of scenes in order, the others have fewer
};

// Primitives per workgroup of the counting and emit kernels of stage 2: a power of two of whole preprocess groups, so that those of
// one workgroup lie in one group of kScanGroup.  Small scenes are short of workgroups, and a workgroup's time is the latency of its steps;
// large ones in no spatial order have so few pairs per workgroup and tile that every pair costs an atomic, fewer the more
// primitives share a workgroup.  Whether there is an order the device knows (in_order); grids are sized for the smaller.  Both kernels, us, 512, 1024, 2048, 4096, 8192 primitives:
//   10 000 at 256 x 256      13.6  15.9  19.9  29.4  48.8      1.2 M inside, ordered   29.2  30.1  32.3  45.8  68.2
//   30 011 at 333 x 217      11.4  12.2  15.0  22.4  35.6      3 M overview, ordered   82.6  59.0  52.1  55.4  63.7
//   500 000 in a cube        90.3  76.5  71.1  75.1  96.1      20 M of a city           823   601   451   373   340
// and all of stage 2: 60 000 in a cube 37.6 37.4 43.2 55.9 73.0, 250 000 61.0 60.8 59.0 72.2 93.7, in order 49.2 47.3 55.8 73.6 94.5; 3 M of
// a city 163 128 111 98 100; 6 M 278 217 173 155 140, in order 99 85 81 89 105.  Images of more than kLdsTilesLarge tiles, whose primitives are
// listed and not counted, have little of either: with 2048 and 8192, 6 M at 4096 x 2304, all of stage 2, city 1381 1364, in order 1339 1357; inside 621
// 607, in order 583 594.
constexpr u32 kBinBlockMax = 8192, kLookForOrder = 2000000, kLookGroups = 32;
static_assert(kScanGroup % (kBinBlockMax / kPreBlock) == 0, "the blocks of one counting workgroup lie in one group");
__host__ __device__ __forceinline__ u32 bin_block(u32 n, u32 tiles, bool ordered)
{
    if (tiles <= kLdsTilesSmall && n <= (ordered ? 1u << 17 : 1u << 16)) return 512u;
    if (tiles <= kLdsTilesSmall && n <= (ordered ? 1u << 18 : 1u << 17)) return 1024u;
    return ordered || n < kLookForOrder ? 2048u : (n < 5000000u ? 4096u : kBinBlockMax);
}

// Are the primitives in spatial order?  With an index they are.  Without, where the workgroups for no order are the wrong ones for an order that
// nobody told of, stage 1 looks: from kLookForOrder primitives on (bin_sort alone, us, with these workgroups and with those for order: 3 M
// inside 98 and 80, 6 M inside 137 and 82, 3 M of a city 67 and 60, 6 M 102 and 78, 6 M overview 269 and 256, 4 M at 640 x 480 281 and
// 285) in images of up to kLdsTilesSmall tiles (beyond: 3 M overview at 3840 x 2160 173 and 194, 6 M of a city at 2560 x 1440 114 and 135).
// They are if most of the pairs of primitives 128 apart that are both binned lie within an eighth of the image of one another.  In
// voxel order at least 0.92 of them do, and of runs of 512 or more that belong together 0.8; in no order or as runs of 10 or 64
// 0.1 to 0.3, sorted along one axis up to 0.43.  Too few pairs, nearly all primitives being culled: no.
__host__ __device__ __forceinline__ bool in_order(const ScratchHeader *h, u32 n)
{
    const bool indexed = h->ordered != 0u;
    if (n < kLookForOrder) return indexed;
    const u32 both = (u32)h->looks, near = (u32)(h->looks >> 32);
    return indexed || (both >= 8u && 2u * near > both);
}

// The primitives of counting workgroup b: `count` of them from `beg` on, none behind the last.  The kernels compare distances from `beg` with
// `count`, since positions behind the share may wrap.
struct BinShare { u32 beg, count; };
__host__ __device__ __forceinline__ BinShare bin_share(u32 b, u32 block, u32 n)
{
    const u64 beg = (u64)b * block;
    return { (u32)beg, beg >= n ? 0u : (n - beg < block ? (u32)(n - beg) : block) };
}

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

inline ScratchLayout scratch_layout(u32 n, u64 capacity, u32 tiles)
{
    ScratchLayout L;
    L.pre_blocks = (n + kPreBlock - 1) / kPreBlock;
    const u32 block = bin_block(n, tiles, true);
    L.bin_blocks = (u32)(((u64)n + block - 1) / block);
    size_t o = 0;
    L.header = o;        o += align256(sizeof(ScratchHeader));
    L.tile_count = o;    o += align256(sizeof(u32) * 2 * ((size_t)tiles + 1));
    L.block_sums = o;    o += align256(sizeof(u32) * (size_t)(L.pre_blocks + 1));
    L.block_offsets = o; o += align256(sizeof(u64) * ((size_t)L.pre_blocks + 1));
    L.group_totals = o;  o += align256(sizeof(u64) * ((size_t)L.pre_blocks / kScanGroup + 2));
    L.tile_masks = o;    o += align256(sizeof(u32) * ((size_t)n + 1));
    L.bin_count = o;     o += align256(sizeof(u32) * ((size_t)L.bin_blocks + 1));
    L.tile_cursor = o;   o += align256(sizeof(u32) * ((size_t)tiles + 1));
    L.big_idx = o;       o += align256(sizeof(u32) * ((size_t)n + 1));
    L.order = o;         o += align256(sizeof(u32) * (size_t)(tiles + 1));
    L.classes = o;       o += align256(sizeof(u32) * 8);
    L.spare = o;         o += align256(sizeof(u32) * 2 * (size_t)(capacity / 2048 + 2));
    L.total = o;
    return L;
}

// Camera-derived kernel arguments (host-computed, passed by value).
struct ProjParams {
    lmk_gs_camera cam;
    float lim_x, lim_y;   // guard band on x/z, y/z for the EWA Jacobian
    u32 tiles_x, tiles_y;
    float tau_tab[8];     // binning rule 1: 2 (ln 255 + ln(1 + (k+1)/8)) + 0.01, k = top 3 mantissa bits of opacity
};

// Launchers (each returns the hipError_t of its launches).
// index == nullptr: every primitive is processed; else the voxel filter runs first and the
// per-workgroup decisions are also written to block_visible when that is not nullptr
hipError_t launch_preprocess(const lmk_gs_gaussians &g, const lmk_gs_voxel_index *index, uint8_t *block_visible,
                             const ProjParams &pp, const lmk_gs_projected &out,
                             char *scratch, const ScratchLayout &L, hipStream_t stream);
// the scratch contents lmk_gs_bin_sort expects from lmk_gs_preprocess, recomputed from proj alone
hipError_t launch_rebuild_handover(const lmk_gs_projected &proj, u32 n, const ProjParams &pp,
                                   char *scratch, const ScratchLayout &L, hipStream_t stream);
// out[0] = D, out[1] = status (sign-extended) from the scratch header
hipError_t launch_copy_status(const char *scratch, const ScratchLayout &L, u64 *out, hipStream_t stream);
hipError_t launch_build_cov3d(const lmk_gs_gaussians &g, float *cov3d, hipStream_t stream);
hipError_t launch_bin_sort(const lmk_gs_projected &proj, u32 n, const ProjParams &pp, const lmk_gs_binned &out,
                           char *scratch, const ScratchLayout &L, hipStream_t stream);
hipError_t launch_render(const lmk_gs_projected &proj, const lmk_gs_binned &binned, const ProjParams &pp,
                         float *out_rgb, float *out_T, hipStream_t stream);
hipError_t launch_render_backward(const lmk_gs_projected &proj, u32 n, const lmk_gs_binned &binned,
                                  const ProjParams &pp, const float *grad_rgb, const float *grad_T,
                                  float *grad_feat, hipStream_t stream);
hipError_t launch_preprocess_backward(const lmk_gs_gaussians &g, const ProjParams &pp,
                                      const lmk_gs_projected &proj, const float *grad_feat,
                                      const lmk_gs_gaussian_grads &out, hipStream_t stream);
hipError_t launch_anchor_decode(const lmk_gs_anchors &anchors, const lmk_gs_anchor_decoder &decoder,
                                const float *cam_pos, const u32 *visible, u32 v, const uint8_t *anchor_visible,
                                const lmk_gs_decoded &out, hipStream_t stream);
// visible[i] = the box (lo, hi, reach of the scales) passes the frustum test of the voxel filter
hipError_t launch_box_flags(const float *box, u32 count, const ProjParams &pp, uint8_t *visible, hipStream_t stream);

}  // namespace lmk
