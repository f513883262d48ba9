// What the compositing kernel and its gradient kernel share: the staged form of a list entry, its exponent
// at a pixel, and which 4x4 pixel cells of the tile it can reach with alpha >= 1/255 (the "intersection
// operations for each tile" of Sec. 4.2.1, applied inside the tile).
#ifndef LMK_GS_BLEND_REACH_H
#define LMK_GS_BLEND_REACH_H
#include "lmk_gs_internal.h"

namespace lmk {

// ---- a list entry as the compositing kernels stage it in LDS, and its exponent at a pixel.
// log2(alpha) = lo - 0.5 log2(e) q with q = A dx^2 + 2 B dx dy + C dy^2 (Sec. 2.2 Eq. 10) is not
// evaluated term by term: for a long thin splat the three terms are thousands of times larger than
// their sum, and fp32 rounding of each would move alpha by 1e-3 of its value.  Completing the square,
//   q = A t^2 + (C - B^2 / A) dy^2,   t = dx + (B / A) dy,
// leaves two non-negative terms.  B / A is taken to twice fp32 precision while staging, so that
// C - B^2 / A keeps full relative accuracy however close the conic is to singular; at a pixel, t
// comes out of one fused multiply-add (one rounding, of t itself).
//   geo = { u - X0, v - Y0, A' = -0.5 log2(e) A, -B / A }
//   cop = { -0.5 log2(e) (C - B^2 / A), lo = log2(opacity), r, g }
//   blue
struct StagedEntry { float4 geo, cop; float blue; };

// a = { u, v, A, B }, b = { C, opacity, r, g } of the feature record; (X0, Y0) = the tile's reference point
__device__ __forceinline__ StagedEntry stage_entry(const float4 a, const float4 b, float blue, float X0, float Y0)
{
    const float kL2E = 1.4426950408889634f;
    const float A = a.z, B = a.w, C = b.x;
    const float r0 = B / A;
    const float r_hi = r0 + fmaf(-r0, A, B) / A;            // B / A to the last bit
    const float r_lo = fmaf(-r_hi, A, B) / A;               // and what fp32 cannot hold of it
    const float c2 = fmaf(-r_lo, B, fmaf(-r_hi, B, C));     // C - B^2 / A
    StagedEntry s;
    s.geo = make_float4(a.x - X0, a.y - Y0, -0.5f * kL2E * A, -r_hi);
    s.cop = make_float4(-0.5f * kL2E * c2, __log2f(b.y), b.z, b.w);
    s.blue = blue;
    return s;
}

// log2(alpha) of a staged entry at the pixel from which its centre lies at (dx, dy)
__device__ __forceinline__ float log2_alpha(const float4 geo, const float4 cop, float dx, float dy)
{
    const float t = fmaf(-geo.w, dy, dx);
    return fmaf(geo.z * t, t, fmaf(cop.x * dy, dy, cop.y));
}

// log2(alpha_max) >= log2(1/255) - margin is a reach, i.e. alpha down to 0.99990/255
constexpr float kBlockPass = -7.994353436858858f - 1.5e-4f;

// Upper bound, with the rounding margin folded in, of A' dx^2 + B' dx dy + C' dy^2 over the square [-half, half]^2 about a
// centre from which the splat centre lies at (xs, ys).  tx = -B / A, ty = -B / C.
__device__ __forceinline__ float square_reach(float xs, float ys, float Aq, float Bq, float Cq, float tx, float ty, float half)
{
    auto clamped = [&](float v) { return __builtin_amdgcn_fmed3f(v, -half, half); };
    const float kRelMargin = -2e-6f;    // times (A' ex^2 + C' ey^2) <= 0: covers fp32 rounding of the test
    // candidate 1: x clamped into the square, best y on that vertical line
    const float ex1 = clamped(xs) - xs;
    const float ey1 = clamped(fmaf(ty, ex1, ys)) - ys;
    const float m1 = fmaf(Aq * ex1, ex1, Cq * ey1 * ey1);
    const float p1 = fmaf(Bq * ex1, ey1, m1);
    // candidate 2: y clamped, best x on that horizontal line
    const float ey2 = clamped(ys) - ys;
    const float ex2 = clamped(fmaf(tx, ey2, xs)) - xs;
    const float m2 = fmaf(Aq * ex2, ex2, Cq * ey2 * ey2);
    const float p2 = fmaf(Bq * ex2, ey2, m2);
    return fmaxf(fmaf(m1, kRelMargin, p1), fmaf(m2, kRelMargin, p2));
}

// The cells of an entry whose level is no ellipse in fp32 (a singular conic, a value that is not finite): those where the
// exponent's largest value over the 8x8 block and over the cell passes.  A comparison with NaN does not pass.  B and C are read
// again from the feature record, so that the path that all other entries take keeps its registers.
__device__ __forceinline__ u32 entry_cells_any(const StagedEntry &s, const float4 *__restrict__ feat, u32 index)
{
    const float kL2E = 1.4426950408889634f;
    const float B = feat[(size_t)index * (LMK_GS_FEAT_STRIDE / 4)].w, C = feat[(size_t)index * (LMK_GS_FEAT_STRIDE / 4) + 1].x;
    const float Bq = -kL2E * B, Cq = -0.5f * kL2E * C, ty = -B / C;
    auto passes = [&](float xs, float ys, float half) { return square_reach(xs, ys, s.geo.z, Bq, Cq, s.geo.w, ty, half) + s.cop.y >= kBlockPass; };
    u32 cells = 0;
#pragma unroll 1
    for (u32 k = 0; k < 16; ++k) {
        const float xs = s.geo.x - (float)((k & 2u) * 4u), ys = s.geo.y - (float)((k & 8u));    // from the centre of the block
        const bool pass = passes(xs, ys, 3.5f) && passes(xs - ((k & 1u) ? 2.0f : -2.0f), ys - ((k & 4u) ? 2.0f : -2.0f), 1.5f);
        cells |= pass ? 1u << k : 0u;
    }
    return cells;
}

// ---- the cells a staged entry reaches: bit 4 r + c = the square of the pixel centres of cell (column c, row r)
// holds a point with log2(alpha) >= kBlockPass.  About the splat's centre the points of that level are
//   X = nr Y +- sqrt((L + c2' Y^2) / -A'),   L = lo - kBlockPass, nr = -B / A,
// an ellipse, so a row of cells, a strip of Y, meets it between its leftmost and rightmost points there: the
// ellipse's own, at Y = -+yr, yr = nr sqrt(L A' / (C' c2')), or those at the edge of the strip nearest to them.
// Two square roots a strip then give the columns of all four cells.  A cell too many costs time and one too few
// a wrong pixel, so rounding is given room: 1e-4 of L (the square roots and yr are good to 1e-6, and a point of the
// ellipse stays within the larger one of it), and 1e-6 of every coordinate that enters a sum.
// One lane does this for an entry as it stages it: 150 vector instructions per 64 entries and tile, 250 with the lists,
// where testing them against four 8x8 blocks (the exponent's largest value over a square), then the survivors
// against four 4x4 cells each, took 450: 94.0 M -> 86.6 M per launch forward, 278 M -> 264 M backward (3 M overview).
// Where the level is no ellipse in fp32 the answer is kNoEllipse, and entry_cells_any() has to be asked.
constexpr u32 kNoEllipse = 0x10000u;
__device__ __forceinline__ u32 entry_cells(const StagedEntry &s)
{
    const float du = s.geo.x, dv = s.geo.y, nr = s.geo.w, An = -s.geo.z, cn = -s.cop.x;
    const float L = s.cop.y - kBlockPass;
    const float inv = __builtin_amdgcn_rcpf(An);
    const float level = fmaf(L, 1.0001f, 1e-4f) * inv, bend = cn * inv;
    const float yr = nr * __builtin_amdgcn_sqrtf(L * An * __builtin_amdgcn_rcpf(fmaf(An * nr, nr, cn) * cn));
    const float mx = 1e-6f * fmaf(fabsf(nr), fabsf(dv) + 12.0f, fabsf(du) + 12.0f), my = 1e-6f * (fabsf(dv) + 12.0f);
    // columns: the first cell whose right edge 4 c - 0.5 is not left of the strip's leftmost point, and the one
    // behind the last whose left edge 4 c - 3.5 is not right of the rightmost
    const float lo0 = fmaf(du - mx, 0.25f, 0.125f), hi0 = fmaf(du + mx, 0.25f, 1.875f);
    const float q = 0.25f * nr;
    u32 cells = 0;
#pragma unroll
    for (u32 r = 0; r < 4; ++r) {
        const float y0 = (4.0f * (float)r - 3.5f - my) - dv, y1 = (4.0f * (float)r - 0.5f + my) - dv;
        const float yR = __builtin_amdgcn_fmed3f(yr, y0, y1), yL = __builtin_amdgcn_fmed3f(-yr, y0, y1);
        const float dR = fmaf(-bend * yR, yR, level), dL = fmaf(-bend * yL, yL, level);
        const float hi = fmaf(q, yR, fmaf(0.25f, __builtin_amdgcn_sqrtf(dR), hi0));
        const float lo = fmaf(q, yL, fmaf(-0.25f, __builtin_amdgcn_sqrtf(fmaxf(dL, 0.0f)), lo0));
        const u32 c0 = (u32)__builtin_amdgcn_fmed3f(ceilf(lo), 0.0f, 4.0f), c1 = (u32)__builtin_amdgcn_fmed3f(floorf(hi), 0.0f, 4.0f);
        const u32 row = (1u << c1) - (1u << c0);
        cells |= (dR >= 0.0f ? row : 0u) << (4u * r);       // a strip beyond the ellipse: no point of it there
    }
    // a value that is not finite, and a root of a negative one (L < 0, C' < 0), come through the sum
    const bool sound = bend > 0.0f && level + bend + fabsf(yr) + fabsf(du) + fabsf(dv) < 3.0e38f;
    return sound ? cells : kNoEllipse;
}

// The entries of a staged batch that reach each of the wavefront's four cells, in list order: put(cell, rank, entry)
// per listed one.  s_cells holds the masks of a batch of up to kCellsBatch, zero behind its end; `shift`
// = bit of the wavefront's first cell; `wanted` leaves out whole cells; of cell q what is at or behind limit[q] is left
// out too if LIMITED.
constexpr u32 kCellsBatch = 256;
__device__ __forceinline__ u32 wave_cells_shift(u32 wv) { return (wv >> 1) * 8u + (wv & 1u) * 2u; }
__device__ __forceinline__ u32 cell_bit(u32 q) { return 1u << ((q & 1u) + (q >> 1) * 4u); }
// the cells with a lane left in `alive`; cell q of a wavefront is its lanes 16 q to 16 q + 15
__device__ __forceinline__ u32 cells_alive(u64 alive)
{
    u32 wanted = 0;
#pragma unroll
    for (u32 q = 0; q < 4; ++q)
        if (((alive >> (16u * q)) & 0xffffull) != 0ull) wanted |= cell_bit(q);
    return wanted;
}
template <bool LIMITED, class Put>
__device__ __forceinline__ void list_cells(const unsigned short *s_cells, u32 cnt, u32 shift, u32 wanted, const u32 (&limit)[4],
                                           u32 lane, u32 (&n4)[4], Put &&put)
{
    n4[0] = n4[1] = n4[2] = n4[3] = 0u;
    u32 cells[kCellsBatch / kWave];                         // read together: one trip to LDS, not one per wavefront of entries
#pragma unroll
    for (u32 j = 0; j < kCellsBatch / kWave; ++j) cells[j] = s_cells[j * kWave + lane];
#pragma unroll
    for (u32 j = 0; j < kCellsBatch / kWave; ++j) {
        const u32 c0 = j * kWave;
        if (c0 >= cnt) break;
        const u32 m = (cells[j] >> shift) & wanted;
#pragma unroll
        for (u32 q = 0; q < 4; ++q) {
            const bool pass = (m & cell_bit(q)) != 0u && (!LIMITED || c0 + lane < limit[q]);
            const u64 mask = __builtin_amdgcn_ballot_w64(pass);
            const u32 rank = __builtin_amdgcn_mbcnt_hi((u32)(mask >> 32), __builtin_amdgcn_mbcnt_lo((u32)mask, n4[q]));
            if (pass) put(q, rank, c0 + lane);
            n4[q] += (u32)__builtin_popcountll(mask);
        }
    }
}

// ---- a tile shared by workgroups (tile_work.h): a wavefront per cell, four lanes a pixel, a lane for each of four
// consecutive entries of the list
// lane q's value in all four lanes of a pixel
template <u32 Q>
__device__ __forceinline__ float quad_lane(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), (int)(Q * 0x55u), 0xf, 0xf, true));
}

// A pixel's way through four entries, a = the alpha of this lane's entry, zero where it is not composited: T in front of
// each and behind the last.  A pixel stops where its transmittance would fall below 1e-4; the products only fall, so
// one look at the last of them tells whether any stops (a few steps of a walk), and there the four are taken one by
// one and what is behind the stop is set to zero.
__device__ __forceinline__ void quad_walk(float T, float (&alpha)[4], float (&Tq)[5], bool &done)
{
    Tq[0] = T;
#pragma unroll
    for (u32 q = 0; q < 4; ++q) Tq[q + 1] = fmaf(-Tq[q], alpha[q], Tq[q]);
    if (__builtin_amdgcn_ballot_w64(Tq[4] < 1e-4f) == 0ull) return;        // a pixel that has stopped keeps its T >= 1e-4
#pragma unroll
    for (u32 q = 0; q < 4; ++q) {
        const float a = done ? 0.0f : alpha[q], Tn = fmaf(-Tq[q], a, Tq[q]);
        done = done || Tn < 1e-4f;
        alpha[q] = done ? 0.0f : a;
        Tq[q + 1] = done ? Tq[q] : Tn;
    }
}

// the entries of a staged batch that reach cell `cell` and lie in front of `limit`, in list order; returns how many
template <class Slot, class Put>
__device__ __forceinline__ u32 list_cell(const Slot *s_cells, u32 cnt, u32 cell, u32 limit, u32 lane, Put &&put)
{
    u32 n = 0;
    u32 cells[kCellsBatch / kWave];
#pragma unroll
    for (u32 j = 0; j < kCellsBatch / kWave; ++j) cells[j] = s_cells[j * kWave + lane];
#pragma unroll
    for (u32 j = 0; j < kCellsBatch / kWave; ++j) {
        const u32 c0 = j * kWave;
        if (c0 >= cnt) break;
        const bool pass = ((cells[j] >> cell) & 1u) != 0u && c0 + lane < limit;
        const u64 mask = __builtin_amdgcn_ballot_w64(pass);
        const u32 rank = __builtin_amdgcn_mbcnt_hi((u32)(mask >> 32), __builtin_amdgcn_mbcnt_lo((u32)mask, n));
        if (pass) put(rank, c0 + lane);
        n += (u32)__builtin_popcountll(mask);
    }
    return n;
}

}  // namespace lmk
#endif
