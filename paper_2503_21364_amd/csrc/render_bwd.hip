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
// entries at a time.  Tiles that the image would wait for go another way, see backward_block.
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

namespace lmk {

namespace {

constexpr u32 kBwdThreads = 256, kBwdBatch = 255, kNullSlot = 255;
constexpr u32 kBwdWaves = kBwdThreads / kWave;
typedef unsigned char slot_t;               // a slot of the staged batch
constexpr u32 kBwdStep = 4;                 // list entries walked together
constexpr u32 kBwdList = kBwdBatch + 1u + 2u * kBwdStep;    // a list and the null slots behind it
static_assert(kBwdList % kBwdStep == 0, "lists are read four slots at a time");
constexpr u32 kTurnStride = kWave + 4;      // floats between the four entries of a step in LDS (bank spread)
constexpr u32 kGradComps = 9;               // moments: m x, m y, m x^2, m x y, m y^2, m, then w per channel

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
    double acc[kBwdBatch + 1][kGradComps];
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
// Consecutive lanes take the consecutive components of an entry, so that the atomics of one
// instruction fall into few cache lines (nine lanes per 36-byte record).
__device__ __forceinline__ void flush_entries(u32 cnt, const BwdSpace &s, float *__restrict__ grad_feat)
{
    for (u32 idx = threadIdx.x; idx < cnt * kGradComps; idx += kBwdThreads) {
        const u32 e = idx / kGradComps, c = idx - e * kGradComps;
        const float kLn2 = 0.6931471805599453f;
        const double *rec = s.acc[e];
        double own = rec[c];
        if (c < 5u) {
            const float4 g = s.geo[e];
            const double u = (double)g.x, v = (double)g.y, M = rec[5], mx = u * M - rec[0], my = v * M - rec[1];
            if (c < 2u) {
                const double Aq = (double)g.z, Bq = (double)s.bc[e].x, Cq = (double)s.bc[e].y;
                own = (double)kLn2 * (c == 0u ? 2.0 * Aq * mx + Bq * my : Bq * mx + 2.0 * Cq * my);
            } else {
                // sum m p q' with p, q' in {dx, dy}: p (sum m q') - q'_centre M_p + M_pq
                const double p = c == 4u ? v : u, q = c == 2u ? u : v, mq = c == 2u ? mx : my;
                const double Mp = c == 4u ? rec[1] : rec[0];
                own = p * mq - q * Mp + own;
                own *= c == 3u ? -1.0 : -0.5;
            }
        } else if (c == 5u) {
            own *= (double)__builtin_amdgcn_exp2f(-s.cop[e].y);       // 1 / opacity
        }
        const float v = (float)own;
        if (v != 0.0f) atomicAdd(grad_feat + (size_t)s.id[e] * LMK_GS_FEAT_STRIDE + c, v);
    }
}

__device__ __forceinline__ void backward_tile(
    BwdSpace &s, u32 tile, const u64 *__restrict__ tile_offsets, const u32 *__restrict__ vals,
    const float4 *__restrict__ feat, const BwdParams &bp, const float *__restrict__ grad_rgb,
    const float *__restrict__ grad_T, float *__restrict__ grad_feat)
{
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
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
    if (len == 0u) return;                                          // the same for the whole workgroup
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
    for (u32 base = 0; base < len; base += kBwdBatch) {
        if (__syncthreads_and(done)) break;        // also: everyone is past the previous batch
        const u32 cnt = len - base < kBwdBatch ? len - base : kBwdBatch;
        if (tid < cnt) {
            const StagedEntry se = stage_entry(next.a, next.b, 0.0f, X0, Y0);
            s.geo[tid] = se.geo; s.cop[tid] = se.cop;
            s.cells[tid] = (unsigned short)entry_cells(se, feat, [&] { return next.id; });
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
            float alpha[kBwdStep];
#pragma unroll
            for (u32 q = 0; q < kBwdStep; ++q) {
                const u32 j = (word >> (8u * q)) & 255u;
                const float4 g = s.geo[j];
                const float2 co = *reinterpret_cast<const float2 *>(&s.cop[j]);
                alpha[q] = fminf(0.99f, __builtin_amdgcn_exp2f(log2_alpha(g, make_float4(co.x, co.y, 0.f, 0.f), g.x - ox, g.y - oy)));
            }
#pragma unroll
            for (u32 q = 0; q < kBwdStep; ++q) {
                const float Tn = fmaf(-T, alpha[q], T);
                const bool hit = !done && !(alpha[q] < 1.0f / 255.0f);
                const bool stop = hit && Tn < 1e-4f;
                const bool upd = hit && !stop;
                T = upd ? Tn : T;
                last = upd ? base + 1u + ((word >> (8u * q)) & 255u) : last;
                done = done || stop;
            }
            if (__builtin_amdgcn_ballot_w64(!done) == 0ull) break;     // all 64 pixels stopped
        }
    }
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
    if (max_last == 0) return;

    // ---- pass 2: back to front
    const size_t plane = (size_t)bp.width * bp.height;
    const size_t pix = (size_t)pyi * bp.width + pxi;
    const float gr = inside ? grad_rgb[pix] : 0.0f;
    const float gg = inside ? grad_rgb[plane + pix] : 0.0f;
    const float gb = inside ? grad_rgb[2 * plane + pix] : 0.0f;
    const float gT = (inside && grad_T) ? grad_T[pix] : 0.0f;
    const float gT_end = gT * T_end;
    const bool odd_grad = __builtin_amdgcn_ballot_w64(!(fabsf(gr) + fabsf(gg) + fabsf(gb) + fabsf(gT_end) < 3.0e38f)) != 0ull;
    float Sr = bp.bg0 * T_end, Sg = bp.bg1 * T_end, Sb = bp.bg2 * T_end;
    T = T_end;
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
    const u32 batches = (max_last + kBwdBatch - 1) / kBwdBatch;
    next = fetch_entry(feat, entry((batches - 1u) * kBwdBatch + tid));
    index = entry(batches > 1u ? (batches - 2u) * kBwdBatch + tid : tid);
    for (u32 b = batches; b-- > 0;) {
        const u32 base = b * kBwdBatch;
        const u32 cnt = max_last - base < kBwdBatch ? max_last - base : kBwdBatch;
        __syncthreads();                // the previous batch has been flushed
        if (tid < cnt) {
            const StagedEntry se = stage_entry(next.a, next.b, next.blue, X0, Y0);
            s.geo[tid] = se.geo; s.cop[tid] = se.cop; s.blue[tid] = se.blue;
            s.bc[tid] = entry_bc(next.a, next.b);
            s.id[tid] = next.id;
            s.cells[tid] = (unsigned short)entry_cells(se, feat, [&] { return next.id; });
            if (!(fabsf(se.cop.z) + fabsf(se.cop.w) + fabsf(se.blue) < 3.0e38f)) s.odd = 1u;
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

// The same for block `block` of a fine tile (see kFineTiles): a wavefront per 4x4 cell, four lanes a pixel, a lane
// for each of four consecutive entries.  Pass 1 is the walk of blend_tile<true>.  In pass 2 a lane has its own
// entry's alpha, 1 / (1 - alpha) and colour; T and the colour S behind go through the four entries back to front, with the
// operations of backward_tile.  m and w are then where
// the matrix instruction wants them: in v_mfma_f64_4x4x4 operand A (entry i, pixel slot k of block b) sits in lane i + 4 b +
// 16 k, that is pixel b + 4 k of the cell; the four blocks' results are added up over the lanes.
// the sum over the lanes of a row of sixteen that agree in lane mod 4, in all of them
__device__ __forceinline__ double row_sum4(double v)
{
    auto turned = [](double x, auto ctrl) {
        const u64 b = (u64)__double_as_longlong(x);
        const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)b, decltype(ctrl)::value, 0xf, 0xf, true);
        const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(b >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return __longlong_as_double((long long)(((u64)hi << 32) | lo));
    };
    v += turned(v, std::integral_constant<int, 0x124>());       // row_ror 4
    return v + turned(v, std::integral_constant<int, 0x128>()); // row_ror 8
}

__device__ __forceinline__ void backward_block(
    BwdSpace &s, u32 tile, u32 block, const u64 *__restrict__ tile_offsets, const u32 *__restrict__ vals,
    const float4 *__restrict__ feat, const BwdParams &bp, const float *__restrict__ grad_rgb,
    const float *__restrict__ grad_T, float *__restrict__ grad_feat)
{
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 pix = lane >> 2, own = lane & 3u;         // pixel of the cell; entry of the four, and moment
    const u32 tx = tile % bp.tiles_x, ty = tile / bp.tiles_x;
    const u32 bi = (block & 1u) * 8u + (wv & 1u) * 4u + (pix & 3u), bj = (block >> 1) * 8u + (wv >> 1) * 4u + (pix >> 2);
    const u32 pxi = tx * LMK_GS_TILE + bi, pyi = ty * LMK_GS_TILE + bj;
    const bool inside = pxi < bp.width && pyi < bp.height;
    const float ox = (float)bi - 3.5f, oy = (float)bj - 3.5f;
    const float X0 = (float)(tx * LMK_GS_TILE) + 4.0f, Y0 = (float)(ty * LMK_GS_TILE) + 4.0f;
    const u32 cell = wave_cells_shift(block) + (wv >> 1) * 4u + (wv & 1u);
    const u64 start = tile_offsets[tile], end = tile_offsets[tile + 1];
    const u64 len64 = end - start;
    const u32 len = len64 < 0xffffff00ull ? (u32)len64 : 0xffffff00u;
    if (len == 0u) return;                              // the same for the whole workgroup
    slot_t *my_list = s.list[wv][0];

    if (tid == kNullSlot) {
        s.geo[kNullSlot] = make_float4(0.f, 0.f, 0.f, 0.f);
        s.cop[kNullSlot] = make_float4(0.f, -1000.0f, 0.f, 0.f);
        s.blue[kNullSlot] = 0.0f;
    }
    // the list of this cell: entries of the staged batch in front of `limit`, null entries behind them
    auto build_list = [&](u32 cnt, u32 limit) -> u32 {
        const u32 n = list_cell(s.cells, cnt, cell, limit, lane, [&](u32 rank, u32 entry) { my_list[rank] = (slot_t)entry; });
        if (lane < 8u) my_list[n + lane] = (slot_t)kNullSlot;
        wave_fence();
        return n;
    };
    auto my_alpha = [&](float4 g, float4 co) { return __builtin_amdgcn_exp2f(log2_alpha(g, co, g.x - ox, g.y - oy)); };

    // ---- pass 1: the forward walk
    float T = 1.0f;
    u32 last = 0;                       // entries of the list up to and including the last composited one
    bool done = !inside;
    const u32 *list = vals + start;
    auto entry = [&](u32 k) { return list[k < len ? k : len - 1u]; };
    u32 index = entry(tid);
    Fetched next = fetch_entry(feat, index);
    index = entry(kBwdBatch + tid);
    for (u32 base = 0; base < len; base += kBwdBatch) {
        if (__syncthreads_and(done)) break;             // also: everyone is past the previous batch
        const u32 cnt = len - base < kBwdBatch ? len - base : kBwdBatch;
        if (tid < cnt) {
            const StagedEntry se = stage_entry(next.a, next.b, 0.0f, X0, Y0);
            s.geo[tid] = se.geo; s.cop[tid] = se.cop;
            s.cells[tid] = (unsigned short)entry_cells(se, feat, [&] { return next.id; });
        } else {
            s.cells[tid] = 0;
        }
        __syncthreads();
        next = fetch_entry(feat, index);
        index = entry(base + 2u * kBwdBatch + tid);
        if (__builtin_amdgcn_ballot_w64(!done) == 0ull) continue;       // this wavefront is finished
        const u32 n = build_list(cnt, kBwdBatch);
        u32 last_k = ~0u;                               // step of the last entry of this lane that the pixel composited
        float4 g, co;
        auto read_step = [&](u32 k) { const u32 e = my_list[k + own]; g = s.geo[e]; co = s.cop[e]; };
        if (n) read_step(0);
        for (u32 k = 0; k < n; k += 4) {
            const float4 g0 = g, co0 = co;
            read_step(k + 4u);                          // while this step is taken; null entries behind the list
            __builtin_amdgcn_sched_barrier(0);
            const float raw = my_alpha(g0, co0);
            const float a = !(raw < 1.0f / 255.0f) && !done ? fminf(0.99f, raw) : 0.0f;
            float alpha[4] = { quad_lane<0>(a), quad_lane<1>(a), quad_lane<2>(a), quad_lane<3>(a) }, Tq[5];
            quad_walk(T, alpha, Tq, done);
            const float mine = own == 0u ? alpha[0] : (own == 1u ? alpha[1] : (own == 2u ? alpha[2] : alpha[3]));
            last_k = mine != 0.0f ? k : last_k;
            T = Tq[4];
            if (__builtin_amdgcn_ballot_w64(!done) == 0ull) break;
        }
        if (last_k != ~0u) last = base + 1u + my_list[last_k + own];
        wave_fence();
    }
    {   // of the pixel, the last of the four
        const u32 t = (u32)__builtin_amdgcn_update_dpp(0, (int)last, 0xB1, 0xf, 0xf, true);
        last = t > last ? t : last;
        const u32 t2 = (u32)__builtin_amdgcn_update_dpp(0, (int)last, 0x4E, 0xf, 0xf, true);
        last = t2 > last ? t2 : last;
    }
    const float T_end = T;

    // the longest walk of this cell and of the tile bound pass 2
    u32 wl = last;
#pragma unroll
    for (int o = 32; o >= 4; o >>= 1) {
        const u32 t = (u32)__shfl_xor((int)wl, o, 64);
        wl = t > wl ? t : wl;
    }
    wl = (u32)__builtin_amdgcn_readfirstlane((int)wl);
    __syncthreads();                    // pass 1 is over in every wavefront: LDS is free
    if (lane == 0) s.last[wv] = wl;
    if (tid == 0) s.odd = 0u;
    __syncthreads();
    u32 max_last = 0;
#pragma unroll
    for (u32 k = 0; k < kBwdWaves; ++k) max_last = s.last[k] > max_last ? s.last[k] : max_last;
    if (max_last == 0) return;

    // ---- pass 2: back to front
    const size_t plane = (size_t)bp.width * bp.height;
    const size_t at = (size_t)pyi * bp.width + pxi;
    const float gr = inside ? grad_rgb[at] : 0.0f;
    const float gg = inside ? grad_rgb[plane + at] : 0.0f;
    const float gb = inside ? grad_rgb[2 * plane + at] : 0.0f;
    const float gT = (inside && grad_T) ? grad_T[at] : 0.0f;
    const float gT_end = gT * T_end;
    const bool odd_grad = __builtin_amdgcn_ballot_w64(!(fabsf(gr) + fabsf(gg) + fabsf(gb) + fabsf(gT_end) < 3.0e38f)) != 0ull;
    float Sr = bp.bg0 * T_end, Sg = bp.bg1 * T_end, Sb = bp.bg2 * T_end;
    T = T_end;
    // operand B (pixel slot k, moment j of block b) sits in lane j + 4 b + 16 k: moment `own` of this lane's pixel
    const double B1 = own == 0u ? 1.0 : (double)(own == 1u ? ox : (own == 2u ? oy : ox * ox));
    const double B2 = own == 0u ? (double)(ox * oy) : (own == 1u ? (double)(oy * oy) : 0.0);
    const double B3 = own == 0u ? (double)gr : (own == 1u ? (double)gg : (own == 2u ? (double)gb : 0.0));
    // a result lane j + 4 b + 16 i adds moment j of instruction b of entry i: components 5, 0, 1, 2 | 3, 4 | 6, 7, 8
    const u32 blk = (lane >> 2) & 3u, ent = lane >> 4;
    const u32 comp = blk == 0u ? (own == 0u ? 5u : own - 1u) : (blk == 1u ? 3u + own : 6u + own);
    const bool adds = blk == 0u || (blk == 1u && own < 2u) || (blk == 2u && own < 3u);
    const u32 batches = (max_last + kBwdBatch - 1) / kBwdBatch;
    next = fetch_entry(feat, entry((batches - 1u) * kBwdBatch + tid));
    index = entry(batches > 1u ? (batches - 2u) * kBwdBatch + tid : tid);
    for (u32 b = batches; b-- > 0;) {
        const u32 base = b * kBwdBatch;
        const u32 cnt = max_last - base < kBwdBatch ? max_last - base : kBwdBatch;
        __syncthreads();                // the previous batch has been flushed
        if (tid < cnt) {
            const StagedEntry se = stage_entry(next.a, next.b, next.blue, X0, Y0);
            s.geo[tid] = se.geo; s.cop[tid] = se.cop; s.blue[tid] = se.blue;
            s.bc[tid] = entry_bc(next.a, next.b);
            s.id[tid] = next.id;
            s.cells[tid] = (unsigned short)entry_cells(se, feat, [&] { return next.id; });
            if (!(fabsf(se.cop.z) + fabsf(se.cop.w) + fabsf(se.blue) < 3.0e38f)) s.odd = 1u;
        } else {
            s.cells[tid] = 0;
        }
        next = fetch_entry(feat, index);
        index = entry(b > 1u ? base - 2u * kBwdBatch + tid : tid);
        for (u32 k = tid; k < cnt * kGradComps; k += kBwdThreads) (&s.acc[0][0])[k] = 0.0;
        __syncthreads();
        const u32 n = base < wl ? build_list(cnt, wl - base) : 0u;
        const u32 my_last = last > base ? last - base : 0u;             // slots below it lie in front of this pixel's end
        const bool odd = odd_grad || s.odd != 0u;                       // wave-uniform
        u32 e1, slot1;
        float4 g1, co1;
        float blue1;
        auto read_step = [&](u32 k) { slot1 = my_list[k + ent]; e1 = my_list[k + own]; g1 = s.geo[e1]; co1 = s.cop[e1]; blue1 = s.blue[e1]; };
        const u32 n_pad = (n + 3u) & ~3u;
        if (n) read_step(n_pad - 4u);
        for (u32 k = n_pad; k > 0;) {
            k -= 4u;
            const u32 e = e1, slot = slot1;
            const float4 g = g1, co = co1;
            const float blue = blue1;
            read_step(k >= 4u ? k - 4u : 0u);           // while this step is taken
            __builtin_amdgcn_sched_barrier(0);
            const float raw = my_alpha(g, co);
            const bool hit = e < my_last && !(raw < 1.0f / 255.0f);     // of fminf(0.99, raw): the same
            const u64 hits = __builtin_amdgcn_ballot_w64(hit);
            if (hits == 0ull) continue;
            // without a contribution everything below is as for a = 0: T and S stay as they are, m and w are zero
            const float a = hit ? fminf(0.99f, raw) : 0.0f;
            const float red = hit ? co.z : 0.0f, green = hit ? co.w : 0.0f, blu = hit ? blue : 0.0f;
            const float inv = __builtin_amdgcn_rcpf(1.0f - a);
            const float T2 = T * quad_lane<3>(inv), T1 = T2 * quad_lane<2>(inv), T0 = T1 * quad_lane<1>(inv), Tf = T0 * quad_lane<0>(inv);
            const float behind = own == 3u ? T : (own == 2u ? T2 : (own == 1u ? T1 : T0));      // transmittance behind this lane's entry
            const float w = a * (own == 3u ? T2 : (own == 2u ? T1 : (own == 1u ? T0 : Tf)));   // ... and in front
            const float w4[4] = { quad_lane<0>(w), quad_lane<1>(w), quad_lane<2>(w), quad_lane<3>(w) };
            T = Tf;
            // the colour behind this lane's entry, and S moved on to in front of the four
            auto behind_own = [&](float c, float &S) {
                const float S2 = fmaf(quad_lane<3>(c), w4[3], S), S1 = fmaf(quad_lane<2>(c), w4[2], S2), S0 = fmaf(quad_lane<1>(c), w4[1], S1);
                const float mine = own == 3u ? S : (own == 2u ? S2 : (own == 1u ? S1 : S0));
                S = fmaf(quad_lane<0>(c), w4[0], S0);
                return mine;
            };
            // dL/da = (dL/dC . (T c - S) - dL/dT_end T_end) / (1 - a); a clamped alpha depends on nothing
            const float num = fmaf(gr, fmaf(behind, red, -behind_own(red, Sr)), fmaf(gg, fmaf(behind, green, -behind_own(green, Sg)),
                              fmaf(gb, fmaf(behind, blu, -behind_own(blu, Sb)), -gT_end)));
            const float m = (raw > 0.99f ? 0.0f : a) * (num * inv);
            const double d1 = row_sum4(__builtin_amdgcn_mfma_f64_4x4x4f64((double)m, B1, 0.0, 0, 0, 0));
            const double d2 = row_sum4(__builtin_amdgcn_mfma_f64_4x4x4f64((double)m, B2, 0.0, 0, 0, 0));
            const double d3 = row_sum4(__builtin_amdgcn_mfma_f64_4x4x4f64((double)w, B3, 0.0, 0, 0, 0));
            // zero times a value that is not finite is NaN: an entry that no pixel of the cell composites adds nothing
            bool add = adds && slot != kNullSlot;
            if (odd) add = add && ((hits >> ent) & 0x1111111111111111ull) != 0ull;
            if (add) atomicAdd(&s.acc[slot][comp], blk == 0u ? d1 : (blk == 1u ? d2 : d3));
        }
        __syncthreads();
        flush_entries(cnt, s, grad_feat);
    }
}

// Workgroups of fine_grid(): the tiles with the longest lists first, when the caller has the hint.
__global__ __launch_bounds__(kBwdThreads, 4) void blend_backward_kernel(
    const u64 *__restrict__ tile_offsets, const u32 *__restrict__ tile_order, const u32 *__restrict__ vals,
    const float4 *__restrict__ feat, BwdParams bp, const float *__restrict__ grad_rgb,
    const float *__restrict__ grad_T, float *__restrict__ grad_feat)
{
    __shared__ BwdSpace space;
    const TileWork w = tile_work(bp.num_tiles, tile_order, tile_offsets, reinterpret_cast<unsigned short *>(space.turn));
    if (w.tile >= bp.num_tiles) return;
    if (w.fine) backward_block(space, w.tile, w.block, tile_offsets, vals, feat, bp, grad_rgb, grad_T, grad_feat);
    else backward_tile(space, w.tile, tile_offsets, vals, feat, bp, grad_rgb, grad_T, grad_feat);
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
    hipLaunchKernelGGL(blend_backward_kernel, dim3(fine_grid(bp.num_tiles, binned.tile_order != nullptr)), dim3(kBwdThreads), 0, stream,
                       binned.tile_offsets, binned.tile_order, binned.vals,
                       reinterpret_cast<const float4 *>(proj.feat), bp, grad_rgb, grad_T, grad_feat);
    return hipGetLastError();
}

}  // namespace lmk
