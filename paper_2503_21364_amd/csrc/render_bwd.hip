// Gradient of a scalar loss through the compositing of stage 3 (Sec. 2.2 Eq. 9-10; the text
// after them: the rasteriser is differentiable and every parameter of the primitives is
// optimised through the rendering process).
//
// For a pixel whose walk composited the entries i = 1..m (T_1 = 1, T_{i+1} = T_i (1 - a_i),
// w_i = a_i T_i, C = sum c_i w_i + bg T_{m+1}), with S_i = sum_{j>i} c_j w_j + bg T_{m+1}:
//   dL/dc_i = w_i dL/dC
//   dL/da_i = dL/dC . (T_i c_i - S_i / (1 - a_i)) - dL/dT_end T_end / (1 - a_i)
//   a = o exp(-q/2), q = A dx^2 + 2 B dx dy + C dy^2:  da/do = a / o, da/dq = -a / 2
// The thresholds of the walk are constants of the derivative: skipped entries, the entry that
// stops the walk and everything behind it get nothing; where a was clamped to 0.99 it depends
// on neither o nor q.
//
// One workgroup per 16x16 tile, one thread per pixel, each wavefront an 8x8 block, each group of 16
// lanes (row) a 4x4 cell of it.  Entries are staged in LDS in batches of 255 (slot 255 is a null
// record that never contributes), with the cells that they can reach (entry_cells, as in blend_kernel).  Per batch
// every wavefront puts the entries of its cells on one list per row; the pixels of a row walk that list, four
// entries at a time.  Tiles that the image would wait for (kSharedTiles) are shared by four workgroups, which take a part of
// the list each, see backward_tile.
// Pass 1 repeats the forward walk with the arithmetic of blend_kernel (same expression for log2(alpha),
// same comparisons), which gives every pixel its final transmittance and the position of its last
// composited entry.  Pass 2 takes the batches, and each list, back to front: T_i is recovered as
// T_{i+1} / (1 - a_i), S_i is a running sum.
//
// What is summed over the pixels of an entry are not the nine gradient components themselves but nine
// moments from which they follow: with m = a dL/da (0 where a was clamped) the sums of m {1, x, y, x^2,
// x y, y^2} over the pixel positions, and of w dL/dC per channel.  Against the four entries of a step the
// pixel's factors -- {1, x, y, x^2}, {x y, y^2} and its upstream gradient -- are constants, so these sums
// are matrix products: (entry x pixel) . (pixel x moment), one 4x4x4 block per row, on the matrix cores in
// double precision (m and w go in as they are, every product is exact, and the positions can be taken
// from the tile's reference point; moving the moments to the splat's centre would lose digits in fp32).
// m and w change from lane = pixel to lane = (entry, pixels) through LDS.  The results are added to
// per-entry LDS accumulators, moved to the splat's centre and multiplied by the per-entry factors (A, B,
// C, 1 / opacity) once per (tile, entry), and leave the workgroup as one global float atomic per (entry,
// component): the order of these additions is not fixed, so results differ from run to run by fp32
// rounding.  A non-finite upstream gradient reaches the entries composited in its row, a non-finite colour
// the pixels that composite it; an infinite one may come out as NaN (the moments are differences).
//
// Bound by vector-instruction issue (the exponent evaluation of the forward pass, twice, and the
// gradient arithmetic) and by the LDS pipe; HBM traffic is the forward's gather, twice, plus 36 bytes of
// atomics per pair.
#include <type_traits>

#include "lmk_gs_internal.h"
#include "blend_reach.h"
#include "tile_work.h"

namespace lmk {

namespace {

constexpr u32 kBwdThreads = 256, kBwdBatch = 255, kNullSlot = 255;
constexpr u32 kBwdWaves = kBwdThreads / kWave;
typedef unsigned char slot_t;               // a slot of the staged batch
constexpr u32 kBwdStep = 4;                 // list entries walked together
constexpr u32 kBwdList = kBwdBatch + 1u + 2u * kBwdStep;    // a list and the null slots behind it
static_assert(kBwdList % kBwdStep == 0, "lists are read four slots at a time");
constexpr u32 kTurnStride = kWave + 4;      // floats between the four entries of a step in LDS (bank spread)
constexpr u32 kParts = 4;                   // workgroups of a tile in parts
// All parts walk the list forwards, so that more lists than this fill the chip with that (30 011 primitives, 131 long lists of 1200, in parts
// 93 us, whole 84; 20 796, 133 of 2016, 76, 65; 104 of 1404 73, 71; 200 000 in a cube, 122 of 306, 150, 170)
constexpr u32 kMostInParts = 128;
constexpr u32 kGradComps = 9;               // moments: m x, m y, m x^2, m x y, m y^2, m, then w per channel

static_assert(kParts * kBwdThreads * 16u <= (kBwdBatch + 1u) * kGradComps * 8u, "what is kept of the segments fits the place of the sums");

struct BwdParams {
    u32 width, height, tiles_x, num_tiles;
    float bg0, bg1, bg2;
};

// B' = -log2(e) B and C' = -0.5 log2(e) C of a fetched entry, for the flush
__device__ __forceinline__ float2 entry_bc(const float4 a, const float4 b)
{
    const float kL2E = 1.4426950408889634f;
    return make_float2(-kL2E * a.w, -0.5f * kL2E * b.x);
}

// one list entry on its way from the feature records to LDS: the index is read two batches ahead and the record one,
// both unconditionally (see fetch_record of the forward pass)
struct Fetched { float4 a, b; float blue; u32 id; };
__device__ __forceinline__ Fetched fetch_entry(const float4 *__restrict__ feat, u32 index)
{
    const float4 *f = feat + (size_t)index * (LMK_GS_FEAT_STRIDE / 4);
    Fetched r;
    r.id = index;
    r.a = f[0]; r.b = f[1]; r.blue = reinterpret_cast<const float *>(f)[8];
    return r;
}

// the four slots at position k of a row's list; beyond the row's own end null slots
__device__ __forceinline__ u32 list_word(const slot_t *list, u32 k, u32 n_pad)
{
    return *reinterpret_cast<const u32 *>(list + (k < n_pad ? k : n_pad));
}

// the staged form of blend_kernel (stage_entry), so that log2(alpha) is evaluated exactly as there
struct BwdSpace {
    float4 geo[kBwdBatch + 1];              // du, dv, A', -B/A
    float4 cop[kBwdBatch + 1];              // -0.5 log2(e) (C - B^2/A), lo, r, g
    float2 bc[kBwdBatch + 1];               // B' = -log2(e) B, C' = -0.5 log2(e) C
    float blue[kBwdBatch + 1];              // b
    u32 id[kBwdBatch + 1];                  // primitive index
    unsigned short cells[kBwdBatch + 1];    // the cells that the entry reaches
    __attribute__((aligned(16))) double acc[kBwdBatch + 1][kGradComps];    // during pass 1 of a tile in parts: what is kept of its segments
    // per wavefront: m (and w) of a step on their way from lane = pixel to lane = (entry, pixels)
    __attribute__((aligned(16))) float turn[kBwdWaves][kBwdStep * kTurnStride];
    __attribute__((aligned(16))) slot_t list[kBwdWaves][4][kBwdList];
    u32 last[kBwdWaves];
    u32 odd;                                // a colour of the list is not finite
};

// From the moments of an entry to its gradient.  About the splat's centre (u, v), seen from the
// reference point: sum m dx = u M - M_x with dx = u - x, and so on; q = A dx^2 + 2 B dx dy + C dy^2,
// da/dq = -a / 2, da/do = a / o; the staged A' = -0.5 log2(e) A, B' = -log2(e) B, C' = -0.5 log2(e) C
// give d/du = ln 2 (2 A' sum m dx + B' sum m dy), d/dv = ln 2 (B' sum m dx + 2 C' sum m dy).
// Lane = entry: its nine results take the place of its sums, as floats.  Then consecutive lanes take the consecutive components of an
// entry, so that the atomics of one instruction fall into few cache lines (nine lanes per 36-byte record).  With both in
// one loop over components every wavefront went through the formulas of all of them nine times, a fifth of the kernel's vector
// instructions: 3 M overview 566 -> 525 us, 500 000 in a cube 375 -> 359, 30 011 at 333 x 217 109 -> 104.
typedef float __attribute__((may_alias)) result_t;
constexpr u32 kResultStride = 2u * kGradComps;
__device__ __forceinline__ void flush_entries(u32 cnt, BwdSpace &s, float *__restrict__ grad_feat)
{
    const u32 tid = threadIdx.x, first = tid & ~(kWave - 1u);
    if (tid < cnt) {
        const double kLn2 = (double)0.6931471805599453f;
        const double *rec = s.acc[tid];
        const float4 g = s.geo[tid];
        const float2 bc = s.bc[tid];
        const double r0 = rec[0], r1 = rec[1], r2 = rec[2], r3 = rec[3], r4 = rec[4], M = rec[5], c0 = rec[6], c1 = rec[7], c2 = rec[8];
        const double u = (double)g.x, v = (double)g.y, Aq = (double)g.z, Bq = (double)bc.x, Cq = (double)bc.y;
        const double mx = u * M - r0, my = v * M - r1;
        result_t *out = reinterpret_cast<result_t *>(s.acc[tid]);
        out[0] = (float)(kLn2 * (2.0 * Aq * mx + Bq * my));
        out[1] = (float)(kLn2 * (Bq * mx + 2.0 * Cq * my));
        // sum m p q' with p, q' in {dx, dy}: p (sum m q') - q'_centre M_p + M_pq
        out[2] = (float)(-0.5 * (u * mx - u * r0 + r2));
        out[3] = (float)(-(u * my - v * r0 + r3));
        out[4] = (float)(-0.5 * (v * my - v * r1 + r4));
        out[5] = (float)(M * (double)__builtin_amdgcn_exp2f(-s.cop[tid].y));      // 1 / opacity
        out[6] = (float)c0; out[7] = (float)c1; out[8] = (float)c2;
    }
    wave_fence();
    const u32 here = cnt > first ? (cnt - first < kWave ? cnt - first : kWave) : 0u;
    const result_t *results = reinterpret_cast<const result_t *>(s.acc[first]);
    for (u32 idx = tid - first; idx < here * kGradComps; idx += kWave) {
        const u32 e = idx / kGradComps, c = idx - e * kGradComps;
        const float v = results[e * kResultStride + c];
        if (v != 0.0f) atomicAdd(grad_feat + (size_t)s.id[first + e] * LMK_GS_FEAT_STRIDE + c, v);
    }
}

// PARTS: part `part` of kParts of the tile's list.  Every workgroup of the tile makes the whole of pass 1, in which it also
// adds up, per segment of the list, the colour that each pixel takes from it; a segment's pass 2 then starts from T behind it
// and the sum of the colours of those behind (sums of terms of one sign, nothing cancels).  So all of an entry's
// pixels are summed in one workgroup, in double, and rounded once, as without parts, and the state that pass 2 starts
// from has fewer roundings than one that was walked back through the whole list (against 64 bits the gradients of a tile of 510
// entries are 1.0e-7 of the sum of their terms' magnitudes off, without parts 1.7e-7; 1020 entries: 1.4e-7, 3.0e-7).  How
// far the walks go is known at the end of pass 1 only: segments are a batch long, and where more than kParts are closed, two
// make one.  Four workgroups then take up to twice the instructions, in half the time or less: by what parts of the tile's
// pixels instead, whose sums meet in fp32, 30 000 primitives at 333 x 217 take 97 us, so 96, and in one piece 140; 1 M in
// clusters at 400 x 300 560, 690, 1184; 200 000 in a cube at 256 x 256 178, 145, 200.
template <bool PARTS>
__device__ __forceinline__ void backward_tile(
    BwdSpace &s, u32 tile, u32 part, const u64 *__restrict__ tile_offsets, const u32 *__restrict__ vals,
    const float4 *__restrict__ feat, const BwdParams &bp, const float *__restrict__ grad_rgb,
    const float *__restrict__ grad_T, float *__restrict__ grad_feat)
{
    u32 tid = threadIdx.x;
    asm volatile("" : "+v"(tid));          // what follows from it is not kept in registers from one work to the next
    const u32 lane = tid & (kWave - 1);
    const u32 wv = (u32)__builtin_amdgcn_readfirstlane((int)(tid / kWave));     // the same for the wavefront: kept in scalar registers
    const u32 tx = tile % bp.tiles_x, ty = tile / bp.tiles_x;
    const u32 grp = lane >> 4, gl = lane & 15u;                    // 4x4 sub-block of the lane, pixel inside it
    const u32 bi = (grp & 1u) * 4u + (gl & 3u), bj = (grp >> 1) * 4u + (gl >> 2);   // pixel inside the 8x8 block
    const u32 pxi = tx * LMK_GS_TILE + (wv & 1u) * 8u + bi, pyi = ty * LMK_GS_TILE + (wv >> 1) * 8u + bj;
    const bool inside = pxi < bp.width && pyi < bp.height;
    // (X0, Y0) = centre of block 0, the reference point of blend_kernel; this block's centre and this
    // lane's pixel centre relative to it
    const float bx = (float)((wv & 1u) * 8u), by = (float)((wv >> 1) * 8u);
    const float ox = bx + ((float)bi - 3.5f), oy = by + ((float)bj - 3.5f);
    const float X0 = (float)(tx * LMK_GS_TILE) + 4.0f, Y0 = (float)(ty * LMK_GS_TILE) + 4.0f;
    const u64 start = tile_offsets[tile], end = tile_offsets[tile + 1];
    const u64 len64 = end - start;
    const u32 len = len64 < 0xffffff00ull ? (u32)len64 : 0xffffff00u;     // a tile's list is far shorter
    if (len == 0u || (PARTS && part * kBwdBatch >= len)) return;    // the same for the whole workgroup
    const u32 cells_shift = wave_cells_shift(wv);
    slot_t *my_list4 = s.list[wv][grp];

    if (tid == kNullSlot) {
        s.geo[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
        s.cop[tid] = make_float4(0.f, -1000.0f, 0.f, 0.f);
        s.blue[tid] = 0.0f;
        s.id[tid] = 0u;
    }
    // lists of the staged batch's first `cnt` entries; returns the longest of the four, n_mine = the length of this row's.
    // limit[q]: slots from there on lie behind the last composited entry of every pixel of cell q
    auto build_lists = [&](auto limited, u32 cnt, u32 wanted, const u32 (&limit)[4], u32 (&n4)[4], u32 &n_mine) -> u32 {
        list_cells<decltype(limited)::value>(s.cells, cnt, cells_shift, wanted, limit, lane, n4,
                                             [&](u32 q, u32 rank, u32 entry) { s.list[wv][q][rank] = (slot_t)entry; });
        n_mine = grp == 0u ? n4[0] : (grp == 1u ? n4[1] : (grp == 2u ? n4[2] : n4[3]));
        if (gl < 2u * kBwdStep) my_list4[n_mine + gl] = (slot_t)kNullSlot;
        wave_fence();
        const u32 l01 = n4[0] > n4[1] ? n4[0] : n4[1], l23 = n4[2] > n4[3] ? n4[2] : n4[3];
        return l01 > l23 ? l01 : l23;
    };

    // ---- pass 1: the forward walk
    float T = 1.0f;
    u32 last = 0;                       // entries of the list up to and including the last composited one
    bool done = !inside;
    const u32 *list = vals + start;
    auto entry = [&](u32 k) { return list[k < len ? k : len - 1u]; };
    u32 index = entry(tid);
    Fetched next = fetch_entry(feat, index);
    index = entry(kBwdBatch + tid);
    // PARTS: the walk so far is up to kParts segments of seg_len batches; of each are kept the colour that it added to the
    // pixel and T behind it
    u32 segs = 0, seg_len = 1, seg_fill = 0;
    float Cr = 0.0f, Cg = 0.0f, Cb = 0.0f;
    float4 *kept = reinterpret_cast<float4 *>(&s.acc[0][0]) + tid;
    auto close_segment = [&] {
        kept[segs * kBwdThreads] = make_float4(Cr, Cg, Cb, T);
        Cr = Cg = Cb = 0.0f;
        ++segs;
        seg_fill = 0;
    };
    for (u32 base = 0; base < len; base += kBwdBatch) {
        if (__syncthreads_and(done)) break;        // also: everyone is past the previous batch
        if (PARTS) {
            if (seg_fill == seg_len) close_segment();
            if (segs == kParts) {                  // two make one
                for (u32 k = 0; k < kParts / 2; ++k) {
                    const float4 a = kept[2 * k * kBwdThreads], b = kept[(2 * k + 1) * kBwdThreads];
                    kept[k * kBwdThreads] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, b.w);
                }
                segs = kParts / 2;
                seg_len *= 2;
            }
            ++seg_fill;
        }
        const u32 cnt = len - base < kBwdBatch ? len - base : kBwdBatch;
        if (tid < cnt) {
            const StagedEntry se = stage_entry(next.a, next.b, PARTS ? next.blue : 0.0f, X0, Y0);
            s.geo[tid] = se.geo; s.cop[tid] = se.cop;
            if (PARTS) s.blue[tid] = se.blue;
            const u32 cells = entry_cells(se);
            s.cells[tid] = (unsigned short)cells;
            if (__builtin_expect(cells == kNoEllipse, 0)) s.cells[tid] = (unsigned short)entry_cells_any(se, feat, next.id);
        } else {
            s.cells[tid] = 0;
        }
        __syncthreads();
        next = fetch_entry(feat, index);
        index = entry(base + 2u * kBwdBatch + tid);
        const u64 alive = __builtin_amdgcn_ballot_w64(!done);
        if (alive == 0ull) continue;                                  // this wavefront is finished
        u32 n4[4], n_mine;
        const u32 no_limit[4] = {};
        const u32 longest = build_lists(std::false_type(), cnt, cells_alive(alive), no_limit, n4, n_mine);
        const u32 n_pad = (n_mine + kBwdStep - 1u) & ~(kBwdStep - 1u);
        for (u32 k = 0; k < longest; k += kBwdStep) {
            const u32 word = list_word(my_list4, k, n_pad);
            float alpha[kBwdStep], colour[kBwdStep][3];
#pragma unroll
            for (u32 q = 0; q < kBwdStep; ++q) {
                const u32 j = (word >> (8u * q)) & 255u;
                const float4 g = s.geo[j];
                const float2 co = *reinterpret_cast<const float2 *>(&s.cop[j]);
                if (PARTS) { colour[q][0] = s.cop[j].z; colour[q][1] = s.cop[j].w; colour[q][2] = s.blue[j]; }
                alpha[q] = fminf(0.99f, __builtin_amdgcn_exp2f(log2_alpha(g, make_float4(co.x, co.y, 0.f, 0.f), g.x - ox, g.y - oy)));
            }
#pragma unroll
            for (u32 q = 0; q < kBwdStep; ++q) {
                const float Tn = fmaf(-T, alpha[q], T);
                const bool hit = !done && !(alpha[q] < 1.0f / 255.0f);
                const bool stop = hit && Tn < 1e-4f;
                const bool upd = hit && !stop;
                if (PARTS) {                        // a colour that is not finite reaches those that composite it
                    const float w = upd ? alpha[q] * T : 0.0f;
                    Cr = fmaf(upd ? colour[q][0] : 0.0f, w, Cr);
                    Cg = fmaf(upd ? colour[q][1] : 0.0f, w, Cg);
                    Cb = fmaf(upd ? colour[q][2] : 0.0f, w, Cb);
                }
                T = upd ? Tn : T;
                last = upd ? base + 1u + ((word >> (8u * q)) & 255u) : last;
                done = done || stop;
            }
            if (__builtin_amdgcn_ballot_w64(!done) == 0ull) break;     // all 64 pixels stopped
        }
    }
    if (PARTS && seg_fill) close_segment();
    const float T_end = T;

    // the longest walk of each sub-block, of each wavefront and of the tile bound pass 2
    u32 wl = last;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        const u32 t = (u32)__shfl_xor((int)wl, o, 64);
        wl = t > wl ? t : wl;
    }
    const u32 sub_last[4] = { (u32)__builtin_amdgcn_readlane((int)wl, 0), (u32)__builtin_amdgcn_readlane((int)wl, 16),
                              (u32)__builtin_amdgcn_readlane((int)wl, 32), (u32)__builtin_amdgcn_readlane((int)wl, 48) };
#pragma unroll
    for (int o = 32; o >= 16; o >>= 1) {
        const u32 t = (u32)__shfl_xor((int)wl, o, 64);
        wl = t > wl ? t : wl;
    }
    __syncthreads();                    // pass 1 is over in every wavefront: LDS is free
    if (lane == 0) s.last[wv] = wl;
    if (tid == 0) s.odd = 0u;
    __syncthreads();
    u32 max_last = 0;
#pragma unroll
    for (u32 k = 0; k < kBwdWaves; ++k) max_last = s.last[k] > max_last ? s.last[k] : max_last;
    // the batches of pass 2, [from, to)
    u32 from = 0, to = (max_last + kBwdBatch - 1) / kBwdBatch;
    if (PARTS) {
        from = part * seg_len;
        to = to < from + seg_len ? to : from + seg_len;
    }
    if (from >= to) return;

    // ---- pass 2: back to front
    const size_t plane = (size_t)bp.width * bp.height;
    const size_t pix = (size_t)pyi * bp.width + pxi;
    const float gr = inside ? grad_rgb[pix] : 0.0f;
    const float gg = inside ? grad_rgb[plane + pix] : 0.0f;
    const float gb = inside ? grad_rgb[2 * plane + pix] : 0.0f;
    const float gT = (inside && grad_T) ? grad_T[pix] : 0.0f;
    const float gT_end = gT * T_end;
    bool odd_grad = __builtin_amdgcn_ballot_w64(!(fabsf(gr) + fabsf(gg) + fabsf(gb) + fabsf(gT_end) < 3.0e38f)) != 0ull;
    float Sr = bp.bg0 * T_end, Sg = bp.bg1 * T_end, Sb = bp.bg2 * T_end;
    if (PARTS) {                        // the state behind the segment
        for (u32 k = segs; k-- > part + 1u;) {
            const float4 c = kept[k * kBwdThreads];
            Sr += c.x; Sg += c.y; Sb += c.z;
        }
        T = kept[part * kBwdThreads].w;
        odd_grad = odd_grad || __builtin_amdgcn_ballot_w64(!(fabsf(Sr) + fabsf(Sg) + fabsf(Sb) < 3.0e38f)) != 0ull;
    }
    // the matrix products.  v_mfma_f64_4x4x4, four blocks: block b = row b of this wavefront; operand A
    // (entry i, pixel slot k) sits in lane i + 4 b + 16 k, operand B (pixel slot k, moment j) in lane
    // j + 4 b + 16 k, the result (entry i, moment j) in lane j + 4 b + 16 i.  In instruction s of four the
    // pixel slot k stands for pixel (x, y) = (s, k) of the sub-block.
    const u32 ml = lane & 3u, mb = (lane >> 2) & 3u, mk = lane >> 4;
    float *turn = s.turn[wv];
    double B1[kBwdStep], B2[kBwdStep], B3[kBwdStep];
    {
        turn[lane] = gr; turn[kWave + lane] = gg; turn[2 * kWave + lane] = gb;
        wave_fence();
        const float my = by + ((float)((mb >> 1) * 4u + mk) - 3.5f);
#pragma unroll
        for (u32 s = 0; s < kBwdStep; ++s) {
            const float mx = bx + ((float)((mb & 1u) * 4u + s) - 3.5f);
            B1[s] = ml == 0u ? 1.0 : (double)(ml == 1u ? mx : (ml == 2u ? my : mx * mx));
            B2[s] = ml == 0u ? (double)(mx * my) : (ml == 1u ? (double)(my * my) : 0.0);
            B3[s] = ml < 3u ? (double)turn[(ml < 3u ? ml : 0u) * kWave + mb * 16u + mk * 4u + s] : 0.0;
        }
        wave_fence();
    }
    const slot_t *out_list = s.list[wv][mb];
    next = fetch_entry(feat, entry((to - 1u) * kBwdBatch + tid));
    index = entry(to > 1u ? (to - 2u) * kBwdBatch + tid : tid);
    for (u32 b = to; b-- > from;) {
        const u32 base = b * kBwdBatch;
        const u32 cnt = max_last - base < kBwdBatch ? max_last - base : kBwdBatch;
        __syncthreads();                // the previous batch has been flushed
        if (tid < cnt) {
            const StagedEntry se = stage_entry(next.a, next.b, next.blue, X0, Y0);
            s.geo[tid] = se.geo; s.cop[tid] = se.cop; s.blue[tid] = se.blue;
            s.bc[tid] = entry_bc(next.a, next.b);
            s.id[tid] = next.id;
            const u32 cells = entry_cells(se);
            s.cells[tid] = (unsigned short)cells;
            if (!(fabsf(se.cop.z) + fabsf(se.cop.w) + fabsf(se.blue) < 3.0e38f)) s.odd = 1u;
            if (__builtin_expect(cells == kNoEllipse, 0)) s.cells[tid] = (unsigned short)entry_cells_any(se, feat, next.id);
        } else {
            s.cells[tid] = 0;
        }
        // the batch in front of this one (all of its slots lie below max_last)
        next = fetch_entry(feat, index);
        index = entry(b > 1u ? base - 2u * kBwdBatch + tid : tid);
        for (u32 k = tid; k < cnt * kGradComps; k += kBwdThreads) (&s.acc[0][0])[k] = 0.0;
        __syncthreads();
        // a wavefront none of whose pixels walked this far has nothing to add (it still takes part
        // in the barriers and the flush below)
        u32 longest = 0, n4[4] = { 0u, 0u, 0u, 0u }, n_mine = 0;
        if (base < wl) {
            u32 limit[4];
#pragma unroll
            for (u32 q = 0; q < 4; ++q) limit[q] = sub_last[q] > base ? sub_last[q] - base : 0u;
            longest = build_lists(std::true_type(), cnt, 0xffffu, limit, n4, n_mine);
        }
        const u32 n_pad = (n_mine + kBwdStep - 1u) & ~(kBwdStep - 1u);
        const u32 n_out = mb == 0u ? n4[0] : (mb == 1u ? n4[1] : (mb == 2u ? n4[2] : n4[3]));
        const u32 out_pad = (n_out + kBwdStep - 1u) & ~(kBwdStep - 1u);
        const u32 my_last = last > base ? last - base : 0u;                 // slots below it lie in front of this pixel's end
        // Zero times a value that is not finite is NaN.  Where such a value is around (ODD), an entry that a pixel
        // does not composite leaves the pixel's S alone, and one that no pixel of a row composites adds nothing for
        // the row; elsewhere both would add zeros and are not asked for.
        auto walk = [&](auto odd_tag) {
            constexpr bool ODD = decltype(odd_tag)::value;
            for (u32 k = (longest + kBwdStep - 1u) & ~(kBwdStep - 1u); k > 0;) {
                k -= kBwdStep;
                const u32 word = list_word(my_list4, k, n_pad);                 // the same for the 16 lanes of a row
                float4 co[kBwdStep];
                float raw[kBwdStep];
                bool hit[kBwdStep], any = false;
#pragma unroll
                for (u32 q = 0; q < kBwdStep; ++q) {
                    const u32 j = (word >> (8u * q)) & 255u;
                    const float4 g = s.geo[j];
                    co[q] = s.cop[j];
                    raw[q] = __builtin_amdgcn_exp2f(log2_alpha(g, co[q], g.x - ox, g.y - oy));
                    hit[q] = j < my_last && !(raw[q] < 1.0f / 255.0f);          // of fminf(0.99, raw): the same
                    any = any || hit[q];
                }
                if (__builtin_amdgcn_ballot_w64(any) == 0ull) continue;          // nothing from this wavefront
                if (ODD) {
#pragma unroll
                    for (u32 q = 0; q < kBwdStep; ++q)
                        if (!hit[q]) co[q].z = co[q].w = 0.0f;
                }
                // a pixel without a contribution goes through the same arithmetic with a = 0: T and S
                // stay as they are and all its moments are zero
                float m[kBwdStep], w[kBwdStep];
#pragma unroll
                for (u32 q = kBwdStep; q-- > 0;) {
                    const float a = hit[q] ? fminf(0.99f, raw[q]) : 0.0f;
                    const float blue = ODD && !hit[q] ? 0.0f : s.blue[(word >> (8u * q)) & 255u];
                    const float inv = __builtin_amdgcn_rcpf(1.0f - a);     // 1 - a >= 0.01; one ulp is enough here
                    // dL/da = (dL/dC . (T c - S) - dL/dT_end T_end) / (1 - a), T = transmittance behind the entry
                    const float num = fmaf(gr, fmaf(T, co[q].z, -Sr), fmaf(gg, fmaf(T, co[q].w, -Sg), fmaf(gb, fmaf(T, blue, -Sb), -gT_end)));
                    T *= inv;                                              // transmittance in front of this entry
                    w[q] = a * T;
                    Sr = fmaf(co[q].z, w[q], Sr); Sg = fmaf(co[q].w, w[q], Sg); Sb = fmaf(blue, w[q], Sb);
                    m[q] = (raw[q] > 0.99f ? 0.0f : a) * (num * inv);      // a dL/da; a clamped alpha depends on nothing
                }
                // lane = pixel -> lane = (entry, row, four pixels); LDS accesses of a wavefront complete in order
#pragma unroll
                for (u32 q = 0; q < kBwdStep; ++q) turn[q * kTurnStride + lane] = m[q];
                wave_fence();
                const float4 am = *reinterpret_cast<const float4 *>(turn + ml * kTurnStride + mb * 16u + mk * 4u);
                wave_fence();
#pragma unroll
                for (u32 q = 0; q < kBwdStep; ++q) turn[q * kTurnStride + lane] = w[q];
                wave_fence();
                const float4 aw = *reinterpret_cast<const float4 *>(turn + ml * kTurnStride + mb * 16u + mk * 4u);
                wave_fence();
                const double Am[kBwdStep] = { (double)am.x, (double)am.y, (double)am.z, (double)am.w };
                const double Aw[kBwdStep] = { (double)aw.x, (double)aw.y, (double)aw.z, (double)aw.w };
                double d1 = 0.0, d2 = 0.0, d3 = 0.0;
#pragma unroll
                for (u32 s = 0; s < kBwdStep; ++s) {
                    d1 = __builtin_amdgcn_mfma_f64_4x4x4f64(Am[s], B1[s], d1, 0, 0, 0);
                    d2 = __builtin_amdgcn_mfma_f64_4x4x4f64(Am[s], B2[s], d2, 0, 0, 0);
                    d3 = __builtin_amdgcn_mfma_f64_4x4x4f64(Aw[s], B3[s], d3, 0, 0, 0);
                }
                // lane j + 4 b + 16 i: moment j of entry i of row b
                u32 slot = out_list[(k < out_pad ? k : out_pad) + mk];
                if (ODD) {
                    u64 hits[kBwdStep];
#pragma unroll
                    for (u32 q = 0; q < kBwdStep; ++q) hits[q] = __builtin_amdgcn_ballot_w64(hit[q]);
                    const u64 h = mk == 0u ? hits[0] : (mk == 1u ? hits[1] : (mk == 2u ? hits[2] : hits[3]));
                    if (((h >> (16u * mb)) & 0xffffull) == 0ull) slot = kNullSlot;
                }
                if (slot != kNullSlot) {
                    double *rec = s.acc[slot];
                    atomicAdd(rec + (ml == 0u ? 5u : ml - 1u), d1);
                    if (ml < 2u) atomicAdd(rec + 3u + ml, d2);
                    if (ml < 3u) atomicAdd(rec + 6u + ml, d3);
                }
            }
        };
        if (odd_grad || s.odd != 0u) walk(std::true_type());                // wave-uniform
        else walk(std::false_type());
        __syncthreads();
        flush_entries(cnt, s, grad_feat);
    }
}

// Workgroups of tile_work_grid(): the tiles with the longest lists first, when the caller has the hint.
__global__ __launch_bounds__(kBwdThreads, 4) void blend_backward_kernel(
    const u64 *__restrict__ tile_offsets, const u32 *__restrict__ tile_order, const u32 *__restrict__ vals,
    const float4 *__restrict__ feat, BwdParams bp, const float *__restrict__ grad_rgb,
    const float *__restrict__ grad_T, float *__restrict__ grad_feat)
{
    __shared__ BwdSpace space;
    const TileWork w = tile_work(blockIdx.x, bp.num_tiles, tile_order, tile_offsets, kMostInParts);
    if (w.shared < bp.num_tiles && tile_offsets[w.shared + 1] - tile_offsets[w.shared] > kBwdBatch) {
        backward_tile<true>(space, w.shared, w.share, tile_offsets, vals, feat, bp, grad_rgb, grad_T, grad_feat);
        return;
    }
    // a list of one batch has no parts
    const u32 whole = w.shared < bp.num_tiles && w.share == 0u ? w.shared : w.whole;
    if (whole < bp.num_tiles) backward_tile<false>(space, whole, 0u, tile_offsets, vals, feat, bp, grad_rgb, grad_T, grad_feat);
}

__global__ __launch_bounds__(256) void zero_kernel(float4 *__restrict__ p, size_t count4)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count4; i += stride)
        p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

}  // namespace

hipError_t launch_render_backward(const lmk_gs_projected &proj, u32 n, const lmk_gs_binned &binned,
                                  const ProjParams &pp, const float *grad_rgb, const float *grad_T,
                                  float *grad_feat, hipStream_t stream)
{
    // a fill kernel, not a memset node: the call may be captured into a graph
    const size_t count4 = (size_t)n * (LMK_GS_FEAT_STRIDE / 4);
    if (count4 > 0) {
        const size_t blocks = (count4 + 255) / 256;
        hipLaunchKernelGGL(zero_kernel, dim3((u32)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, stream,
                           reinterpret_cast<float4 *>(grad_feat), count4);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    BwdParams bp;
    bp.width = pp.cam.width; bp.height = pp.cam.height;
    bp.tiles_x = pp.tiles_x; bp.num_tiles = pp.tiles_x * pp.tiles_y;
    bp.bg0 = pp.cam.bg[0]; bp.bg1 = pp.cam.bg[1]; bp.bg2 = pp.cam.bg[2];
    if (n == 0 || binned.capacity == 0) return hipSuccess;
    hipLaunchKernelGGL(blend_backward_kernel, dim3(tile_work_grid(bp.num_tiles, binned.tile_order != nullptr)), dim3(kBwdThreads), 0, stream,
                       binned.tile_offsets, binned.tile_order, binned.vals,
                       reinterpret_cast<const float4 *>(proj.feat), bp, grad_rgb, grad_T, grad_feat);
    return hipGetLastError();
}

}  // namespace lmk
