// Stage 3: per-tile front-to-back alpha compositing (Sec. 2.2 Eq. 9-10; the
// blend kernel whose share of render time Sec. 4.2.1 reports).
//
// One workgroup (4 wavefronts) per 16x16 tile; each wavefront owns a compact
// 8x8 pixel block, each group of 16 lanes a 4x4 sub-block of it, one pixel per
// lane.  The tile's sorted list is consumed in batches of 256 entries staged in
// LDS (each thread fetches one 48-byte feature record; the next batch's records
// are already in flight while the current batch is composited -- the software
// pipelining of Sec. 4.2.1).
//
// Per batch:
//  1. lane = entry, as it is staged: which of the tile's sixteen 4x4 cells can it reach with
//     alpha >= 1/255?  The exact splat/cell intersection ("intersection operations for each tile",
//     Sec. 4.2.1) from its leftmost and rightmost points in the four rows of cells (entry_cells).
//  2. lane = entry.  Every wavefront puts the entries of each of its four cells on a list, in list
//     order (ballot + mbcnt ranks).  A splat that reaches an 8x8 block touches on average only about
//     half of its cells, and the vector units -- the bound of this kernel -- are spent on (pixel,
//     splat) pairs that can contribute.
//  3. lane = pixel.  Each group walks its own list, four entries at a time: one
//     16-byte LDS read yields four record offsets, the four exponentials are
//     independent, the compositing updates follow in order under per-lane
//     select masks.  The loop runs to the longest of the four lists (shorter
//     ones read a null record) and has no data-dependent scalar control flow
//     (the scalar unit, shared by the CU's four SIMDs, was as loaded as the
//     vector units when survivors were walked with scalar bit scans).
// A wavefront whose 64 pixels have all stopped skips the rest (per-wavefront
// progress, Sec. 4.2.1); the tile leaves when all four have.  Bound by FP32
// VALU issue; HBM traffic is the 52 bytes per list entry of the gather.
#include "lmk_gs_internal.h"
#include "blend_reach.h"
#include "tile_work.h"

namespace lmk {

constexpr u32 kBlendThreads = 256;
constexpr u32 kBatch = 256;
constexpr u32 kXcds = 8;     // MI355X: 8 accelerator dies, workgroups are dealt to them round-robin

constexpr u32 kSurv = 4;     // survivors evaluated together (independent exponentials in flight)

struct BlendParams {
    u32 width, height, tiles_x, num_tiles, tiles_per_xcd;
    float bg0, bg1, bg2;
};

// A list entry on its way from the feature records to LDS.  The two dependent reads, index and record, are each a batch
// ahead of what needs them, and unconditional (a thread beyond the end of the list reads its last entry again): behind
// a branch the compiler waits for what it loads at once, a trip to memory each and batch (3 M overview, 1080p: frame
// 451 -> 442 us, gradient 569 -> 549).
struct Rec { float4 a, b; float blue; };

__device__ __forceinline__ Rec fetch_record(const float4 *__restrict__ feat, u32 index)
{
    const float4 *f = feat + (size_t)index * (LMK_GS_FEAT_STRIDE / 4);
    Rec r;
    r.a = f[0]; r.b = f[1]; r.blue = reinterpret_cast<const float *>(f)[8];
    return r;
}

constexpr u32 kListLen = kBatch + 8;    // survivors of a batch plus null padding

// The staged form of a batch's entries (stage_entry): (du, dv) = splat centre relative to the centre of
// block 0 and the coefficients of log2(alpha) with the square completed.  Slot kBatch is a null record that
// can never contribute.
struct BlendSpace {
    float4 geo[kBatch + 1];     // du, dv, A', -B/A
    float4 cop[kBatch + 1];     // -0.5 log2(e) (C - B^2/A), lo, r, g
    float4 blue[kBatch + 1];    // b: one word, at the offset of the others
    unsigned short cells[kBatch];       // the cells that the entry reaches
    // the cells' lists hold the records' byte offsets inside geo / cop / blue (at most 4096)
    __attribute__((aligned(16))) unsigned short list[kBlendThreads / kWave][4][kListLen];
};

// SHARED: workgroup `block` of four of the tile, a wavefront per cell (see tile_work.h).  A lane evaluates one of four
// entries; all four lanes then take the pixel through the four in order, with the operations of the other form,
// and add up a colour channel each.
template <bool SHARED>
__device__ __forceinline__ void blend_tile(
    BlendSpace &s, u32 tile, u32 block, const u64 *__restrict__ tile_offsets, const u32 *__restrict__ vals,
    const float4 *__restrict__ feat, const BlendParams &bp, float *__restrict__ out_rgb, float *__restrict__ out_T)
{
    u32 tid = threadIdx.x;
    asm volatile("" : "+v"(tid));          // what follows from it is not kept in registers from one work to the next
    const u32 lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 tx = tile % bp.tiles_x, ty = tile / bp.tiles_x;
    // cell and pixel inside it of this lane: its group of 16 and place there, or its wavefront and group of 4
    const u32 grp = SHARED ? wv : lane >> 4, gl = SHARED ? lane >> 2 : lane & 15u, own = lane & 3u;
    const u32 quarter = SHARED ? block : wv;                      // the 8x8 block
    const u32 bi = (quarter & 1u) * 8u + (grp & 1u) * 4u + (gl & 3u), bj = (quarter >> 1) * 8u + (grp >> 1) * 4u + (gl >> 2);
    const u32 pxi = tx * LMK_GS_TILE + bi, pyi = ty * LMK_GS_TILE + bj;     // (bi, bj) = pixel inside the tile
    const bool inside = pxi < bp.width && pyi < bp.height;
    const float ox = (float)bi - 3.5f, oy = (float)bj - 3.5f;
    const float X0 = (float)(tx * LMK_GS_TILE) + 4.0f, Y0 = (float)(ty * LMK_GS_TILE) + 4.0f;
    const u32 cells_shift = SHARED ? wave_cells_shift(block) + (wv >> 1) * 4u + (wv & 1u) : wave_cells_shift(wv);
    const char *geo = reinterpret_cast<const char *>(s.geo), *cop = reinterpret_cast<const char *>(s.cop);
    const char *blu = reinterpret_cast<const char *>(s.blue);
    const char *channel = own < 2u ? cop + 8u + 4u * own : blu;             // SHARED: of this lane (none for the last of the four)

    const u64 start = tile_offsets[tile], end = tile_offsets[tile + 1];
    float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;           // SHARED: channel `own` in cr
    bool done = !inside;
    constexpr u32 kNullOfs = kBatch * 16u;

    if (tid == 0) {
        s.geo[kBatch] = make_float4(0.f, 0.f, 0.f, 0.f);
        s.cop[kBatch] = make_float4(0.f, -1000.0f, 0.f, 0.f);
        s.blue[kBatch].x = 0.0f;
    }
    if (start < end) {                                          // the same for the workgroup
        const u32 *list = vals + start;
        const u32 len = (u32)(end - start);
        auto entry = [&](u32 k) { return list[k < len ? k : len - 1u]; };
        u32 index = entry(tid);
        Rec next = fetch_record(feat, index);
        index = entry(kBatch + tid);

        for (u32 base = 0; base < len; base += kBatch) {
            if (__syncthreads_and(done)) break;        // also: everyone is past the previous batch
            const u32 cnt = len - base < kBatch ? len - base : kBatch;
            {
                // every thread stages one slot; slots past the end of the list reach nothing
                const bool valid = tid < cnt;
                const StagedEntry se = stage_entry(next.a, next.b, next.blue, X0, Y0);
                const u32 cells = valid ? entry_cells(se) : 0u;
                s.geo[tid] = valid ? se.geo : make_float4(0.f, 0.f, 0.f, 0.f);
                s.cop[tid] = valid ? se.cop : make_float4(0.f, -1000.0f, 0.f, 0.f);
                s.blue[tid].x = valid ? se.blue : 0.0f;
                s.cells[tid] = (unsigned short)cells;
                if (__builtin_expect(cells == kNoEllipse, 0)) s.cells[tid] = (unsigned short)entry_cells_any(se, feat, entry(base + tid));
            }
            __syncthreads();
            next = fetch_record(feat, index);                          // in flight during the loops below
            index = entry(base + 2u * kBatch + tid);
            const u64 alive = __builtin_amdgcn_ballot_w64(!done);
            if (alive == 0ull) continue;                               // this wavefront is finished

            if (SHARED) {
                unsigned short *my_list = s.list[wv][0];
                const u32 n = list_cell(s.cells, cnt, cells_shift, kBatch, lane, [&](u32 rank, u32 entry) { my_list[rank] = (unsigned short)(entry * 16u); });
                if (lane < 8u) my_list[n + lane] = (unsigned short)kNullOfs;
                wave_fence();
                // the records of a step are read while the step before it is taken
                struct Step { float4 g; float2 co; float c[4]; } next_step;
                auto read_step = [&](u32 k) {
                    const uint2 four = *reinterpret_cast<const uint2 *>(my_list + k);
                    const u32 mine = my_list[k + own];
                    const u32 lo = (u32)__builtin_amdgcn_readfirstlane((int)four.x), hi = (u32)__builtin_amdgcn_readfirstlane((int)four.y);
                    const u32 ofs[4] = { lo & 0xffffu, lo >> 16, hi & 0xffffu, hi >> 16 };
                    next_step.g = *reinterpret_cast<const float4 *>(geo + mine);
                    next_step.co = *reinterpret_cast<const float2 *>(cop + mine);
    #pragma unroll
                    for (u32 q = 0; q < 4; ++q) next_step.c[q] = *reinterpret_cast<const float *>(channel + ofs[q]);
                };
                if (n) read_step(0);
                for (u32 k = 0; k < n; k += 4) {
                    const Step st = next_step;
                    read_step(k + 4u);                              // null records behind the list
                    __builtin_amdgcn_sched_barrier(0);
                    const float raw = __builtin_amdgcn_exp2f(log2_alpha(st.g, make_float4(st.co.x, st.co.y, 0.f, 0.f), st.g.x - ox, st.g.y - oy));
                    const float a = !(raw < 1.0f / 255.0f) && !done ? fminf(0.99f, raw) : 0.0f;
                    float alpha[4] = { quad_lane<0>(a), quad_lane<1>(a), quad_lane<2>(a), quad_lane<3>(a) }, Tq[5];
                    quad_walk(T, alpha, Tq, done);
    #pragma unroll
                    for (u32 q = 0; q < 4; ++q) cr = fmaf(st.c[q], alpha[q] * Tq[q], cr);
                    T = Tq[4];
                    if (__builtin_amdgcn_ballot_w64(!done) == 0ull) break;
                }
                wave_fence();
                continue;
            }

            // ---- the lists of this wavefront's four cells; a cell whose pixels have all stopped takes nothing more
            u32 n4[4];
            const u32 no_limit[4] = {};
            list_cells<false>(s.cells, cnt, cells_shift, cells_alive(alive), no_limit, lane, n4,
                              [&](u32 q, u32 rank, u32 entry) { s.list[wv][q][rank] = (unsigned short)(entry * 16u); });
            const u32 n_mine = grp == 0u ? n4[0] : (grp == 1u ? n4[1] : (grp == 2u ? n4[2] : n4[3]));
            const u32 l01 = n4[0] > n4[1] ? n4[0] : n4[1], l23 = n4[2] > n4[3] ? n4[2] : n4[3];
            const u32 longest = (u32)__builtin_amdgcn_readfirstlane((int)(l01 > l23 ? l01 : l23));
            unsigned short *my_list = s.list[wv][grp];
            // null records behind every list: a group past its own end keeps reading these
            if (gl < 8u) my_list[n_mine + gl] = (unsigned short)kNullOfs;
            const u32 n4_pad = (n_mine + kSurv - 1u) & ~(kSurv - 1u);

            // ---- lane = pixel; composite the cell's entries in list order, kSurv at a time
            for (u32 k = 0; k < longest; k += kSurv) {
                const uint2 ofs4 = *reinterpret_cast<const uint2 *>(my_list + (k < n4_pad ? k : n4_pad));
                const u32 ofs[kSurv] = { ofs4.x & 0xffffu, ofs4.x >> 16, ofs4.y & 0xffffu, ofs4.y >> 16 };
                // all reads of the four records in flight together: left to itself the compiler waits for one after the other
                float alpha[kSurv], blue[kSurv];
                float4 g[kSurv], co[kSurv];
    #pragma unroll
                for (u32 q = 0; q < kSurv; ++q) {
                    g[q] = *reinterpret_cast<const float4 *>(geo + ofs[q]);
                    co[q] = *reinterpret_cast<const float4 *>(cop + ofs[q]);
                }
    #pragma unroll
                for (u32 q = 0; q < kSurv; ++q) blue[q] = *reinterpret_cast<const float *>(blu + ofs[q]);
                __builtin_amdgcn_sched_barrier(0);
    #pragma unroll
                for (u32 q = 0; q < kSurv; ++q)
                    alpha[q] = fminf(0.99f, __builtin_amdgcn_exp2f(log2_alpha(g[q], co[q], g[q].x - ox, g[q].y - oy)));
    #pragma unroll
                for (u32 q = 0; q < kSurv; ++q) {
                    const float Tn = fmaf(-T, alpha[q], T);
                    const bool hit = !(alpha[q] < 1.0f / 255.0f) && !done;
                    const bool stop = hit && Tn < 1e-4f;
                    const bool upd = hit && !stop;
                    const float w = upd ? alpha[q] * T : 0.0f;
                    cr = fmaf(co[q].z, w, cr); cg = fmaf(co[q].w, w, cg); cb = fmaf(blue[q], w, cb);
                    T = upd ? Tn : T;
                    done = done || stop;
                }
                if (__builtin_amdgcn_ballot_w64(!done) == 0ull) break;     // all 64 pixels stopped
            }
        }
    }
    if (inside) {
        const size_t plane = (size_t)bp.width * bp.height;
        const size_t p = (size_t)pyi * bp.width + pxi;
        if (SHARED) {
            float *dst = own == 3u ? out_T : out_rgb + own * plane;
            dst[p] = own == 3u ? T : cr + T * (own == 0u ? bp.bg0 : (own == 1u ? bp.bg1 : bp.bg2));
        } else {
            out_rgb[p] = cr + T * bp.bg0;
            out_rgb[plane + p] = cg + T * bp.bg1;
            out_rgb[2 * plane + p] = cb + T * bp.bg2;
            out_T[p] = T;
        }
    }
}

// Workgroups of tile_work_grid(): with the caller's order the tiles with the longest lists start first, and consecutive
// workgroup ids, dealt round-robin to the dies, spread them; without it each die gets one contiguous band of
// tiles, so that neighbouring tiles share its L2.
__global__ __launch_bounds__(kBlendThreads, 6) void blend_kernel(
    const u64 *__restrict__ tile_offsets, const u32 *__restrict__ tile_order,
    const u32 *__restrict__ vals, const float4 *__restrict__ feat, BlendParams bp,
    float *__restrict__ out_rgb, float *__restrict__ out_T)
{
    __shared__ BlendSpace space;
    TileWork w;
    if (!tile_order && bp.num_tiles > kSharedTiles) {
        const u32 tile = (blockIdx.x % kXcds) * bp.tiles_per_xcd + blockIdx.x / kXcds;
        w = { blockIdx.x / kXcds < bp.tiles_per_xcd && tile < bp.num_tiles ? tile : bp.num_tiles, bp.num_tiles, 0u };
    } else {
        w = tile_work(blockIdx.x, bp.num_tiles, tile_order, tile_offsets);
    }
    if (w.whole < bp.num_tiles) blend_tile<false>(space, w.whole, 0u, tile_offsets, vals, feat, bp, out_rgb, out_T);
    else if (w.shared < bp.num_tiles) blend_tile<true>(space, w.shared, w.share, tile_offsets, vals, feat, bp, out_rgb, out_T);
}

hipError_t launch_render(const lmk_gs_projected &proj, const lmk_gs_binned &binned, const ProjParams &pp,
                         float *out_rgb, float *out_T, hipStream_t stream)
{
    BlendParams bp;
    bp.width = pp.cam.width; bp.height = pp.cam.height;
    bp.tiles_x = pp.tiles_x; bp.num_tiles = pp.tiles_x * pp.tiles_y;
    bp.tiles_per_xcd = (bp.num_tiles + kXcds - 1) / kXcds;
    bp.bg0 = pp.cam.bg[0]; bp.bg1 = pp.cam.bg[1]; bp.bg2 = pp.cam.bg[2];
    const bool listed = binned.tile_order || bp.num_tiles <= kSharedTiles;
    const u32 grid = listed ? tile_work_grid(bp.num_tiles, binned.tile_order != nullptr) : bp.tiles_per_xcd * kXcds;
    hipLaunchKernelGGL(blend_kernel, dim3(grid), dim3(kBlendThreads), 0, stream,
                       binned.tile_offsets, binned.tile_order, binned.vals,
                       reinterpret_cast<const float4 *>(proj.feat), bp, out_rgb, out_T);
    return hipGetLastError();
}

}  // namespace lmk
