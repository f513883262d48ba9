// Binning rule 1 (lmk_gs_camera.binning == 1; the per-tile intersection test of Sec. 4.2.1): can
// the splat reach alpha >= 1/255 on the square spanned by a tile's pixel centres?
// q(d) = d^T conic d is convex: its minimum over the square is at the splat centre if that is
// inside, else on an edge facing it (clamp one coordinate, minimise along that line; two
// candidates cover all cases).  Contributing needs q <= 2 ln(255 o); tau bounds that from above
// from the exponent and the top three mantissa bits of o (table from the host), so no run-time
// logarithm decides an integer.  Every translation unit that includes this header is compiled
// without floating-point contraction and with correctly rounded division: the projection kernel
// counts the kept tiles, the binning kernels enumerate them, and both must take every decision
// alike (and like the CPU definition of the rule, which runs the same fp32 operation sequence).
#ifndef LMK_GS_TILE_TEST_H
#define LMK_GS_TILE_TEST_H
#include "lmk_gs_internal.h"

namespace lmk {

struct TileTest { float u, v, A, B, C, rx, ry, tau; };

__device__ __forceinline__ float opacity_tau(const ProjParams &pp, float o)
{
    const u32 bits = __float_as_uint(o);
    const int E = (int)((bits >> 23) & 0xffu) - 127;
    return pp.tau_tab[(bits >> 20) & 7u] + (float)E * 1.3862944f;
}

__device__ __forceinline__ TileTest make_tile_test(float u, float v, float A, float B, float C, float tau)
{
    TileTest t;
    t.u = u; t.v = v; t.A = A; t.B = B; t.C = C; t.tau = tau;
    t.rx = -B / A; t.ry = -B / C;
    return t;
}

__device__ __forceinline__ float clampf3(float v, float lo, float hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ __forceinline__ float quad_adj(const TileTest &t, float ex, float ey)
{
    const float m = t.A * ex * ex + t.C * ey * ey;
    const float q = m + 2.0f * t.B * ex * ey;
    return q - 4e-6f * m;
}

// the least q (less a margin for rounding) on the square of a tile's pixel centres
__device__ __forceinline__ float tile_reach(const TileTest &t, u32 tx, u32 ty)
{
    const float h = 0.5f * (float)LMK_GS_TILE - 0.5f;
    const float xs = t.u - ((float)(tx * LMK_GS_TILE) + 0.5f * (float)LMK_GS_TILE);
    const float ys = t.v - ((float)(ty * LMK_GS_TILE) + 0.5f * (float)LMK_GS_TILE);
    const float ex1 = clampf3(xs, -h, h) - xs;
    const float ey1 = clampf3(ys + t.ry * ex1, -h, h) - ys;
    const float ey2 = clampf3(ys, -h, h) - ys;
    const float ex2 = clampf3(xs + t.rx * ey2, -h, h) - xs;
    const float q1 = quad_adj(t, ex1, ey1);
    const float q2 = quad_adj(t, ex2, ey2);
    return q1 < q2 ? q1 : q2;
}
__device__ __forceinline__ bool tile_kept(const TileTest &t, u32 tx, u32 ty) { return tile_reach(t, tx, ty) <= t.tau; }

// How many of the tiles x0 <= tx < x1 of row ty are kept, as tile_kept decides them, but asked only where that is not
// certain.  A tile is kept where its square meets the ellipse q = tau, and in a row of tiles, a strip of y, the ellipse lies
// between its leftmost and rightmost points there: two square roots give the columns.  M bounds A x^2 + C y^2 over the rectangle,
// `slack` is 2e-5 M.  tile_reach is within 5e-6 M of the least q of a tile, and the ends in here are those of an ellipse that differs by as
// little (cn and the products by some 1e-6 M in q, an end by 2e-6 of the rectangle's distance, which is 6e-6 M), so that the ellipse of
// tau - 2 slack holds no tile that is not kept, and beyond that of tau + 2 slack none is.  Where the numbers are no ellipse all
// are asked.
__device__ __forceinline__ u32 row_kept(const TileTest &t, u32 ty, u32 x0, u32 x1, float slack)
{
    const float TS = (float)LMK_GS_TILE, h = 0.5f * TS - 0.5f;
    const float xc = ((float)(x0 * LMK_GS_TILE) + 0.5f * TS) - t.u, yc = ((float)(ty * LMK_GS_TILE) + 0.5f * TS) - t.v;   // centre of the first tile
    const float y0 = yc - h, y1 = yc + h, lo0 = (-h - xc) / TS, hi0 = (h - xc) / TS + 1.0f, wide = (float)(x1 - x0);
    const float cn = t.C + t.B * t.rx, inv = __builtin_amdgcn_rcpf(t.A), bend = t.A * __builtin_amdgcn_rcpf(t.C * cn);
    auto inside = [&](float level, u32 &first, u32 &end) {
        const float yr = t.rx * __builtin_amdgcn_sqrtf(fmaxf(level * bend, 0.0f));      // row of the rightmost point; the leftmost's is -yr
        const float yR = __builtin_amdgcn_fmed3f(yr, y0, y1), yL = __builtin_amdgcn_fmed3f(-yr, y0, y1);
        const float dR = (level - cn * yR * yR) * inv, dL = (level - cn * yL * yL) * inv;
        const float right = t.rx * yR + __builtin_amdgcn_sqrtf(fmaxf(dR, 0.0f)), left = t.rx * yL - __builtin_amdgcn_sqrtf(fmaxf(dL, 0.0f));
        first = (u32)__builtin_amdgcn_fmed3f(ceilf(left / TS + lo0), 0.0f, wide);
        end = dR >= 0.0f ? (u32)__builtin_amdgcn_fmed3f(floorf(right / TS + hi0), 0.0f, wide) : 0u;
    };
    u32 a, b, sure_a, sure_b, kept = 0;
    inside(t.tau + 2.0f * slack, a, b);
    inside(t.tau - 2.0f * slack, sure_a, sure_b);
    if (!(t.A > 0.0f && cn > 0.0f && slack + inv + fabsf(bend) + fabsf(t.rx) + fabsf(t.tau) < 3.0e38f)) { a = 0u; b = x1 - x0; sure_b = 0u; }
    if (sure_a < a) sure_a = a;
    if (sure_b > b) sure_b = b;
    if (sure_b <= sure_a) sure_a = sure_b = b;                  // none is sure
    kept = sure_b - sure_a;
    for (; a < sure_a; ++a) kept += tile_kept(t, x0 + a, ty) ? 1u : 0u;
    for (; sure_b < b; ++sure_b) kept += tile_kept(t, x0 + sure_b, ty) ? 1u : 0u;
    return kept;
}

// The tiles of a bin of kBinEdge x kBinEdge, bit kBinEdge j + i = tile (bx + i, by + j): those that tile_kept surely keeps, and those that have
// to be asked.  A tile is kept where its square meets the ellipse q = tau, and in a row of tiles, a strip of y, the ellipse
// lies between its leftmost and rightmost points there (as in row_kept), so two square roots a row give the columns.  M
// bounds A x^2 + C y^2 over the bin.  tile_reach is within 5e-6 M of the least q of a tile, and the ends in here are those of an
// ellipse that differs by as little (cn and the products by some 1e-6 M in q, an end by 2e-6 of the bin's distance, which is 6e-6 M), so
// that the ellipse of tau - slack, slack = 4e-5 M, holds no tile that is not kept, and beyond that of tau + slack none
// is (over the random ellipses of tests/host/bin_tiles_driver.cpp none is wrong down to 5e-6 M).  Where the numbers are no
// ellipse all are to be asked.
constexpr u32 kBinEdge = 4, kBinTiles = kBinEdge * kBinEdge;
__device__ __forceinline__ void bin_tiles(const TileTest &t, u32 bx, u32 by, u32 &sure, u32 &open)
{
    const float TS = (float)LMK_GS_TILE, h = 0.5f * TS - 0.5f, span = (float)((kBinEdge - 1u) * LMK_GS_TILE);
    const float xc = ((float)(bx * LMK_GS_TILE) + 0.5f * TS) - t.u, yc = ((float)(by * LMK_GS_TILE) + 0.5f * TS) - t.v;   // centre of the first tile
    const float fx = fmaxf(fabsf(xc - h), fabsf(xc + (span + h))), fy = fmaxf(fabsf(yc - h), fabsf(yc + (span + h)));
    const float slack = 4e-5f * (t.A * fx * fx + t.C * fy * fy);
    const float cn = t.C + t.B * t.rx, inv = __builtin_amdgcn_rcpf(t.A), bend = t.A * __builtin_amdgcn_rcpf(t.C * cn);
    const float lo0 = (-h - xc) / TS, hi0 = (h - xc) / TS + 1.0f;
    auto inside = [&](float level) -> u32 {
        const float yr = t.rx * __builtin_amdgcn_sqrtf(fmaxf(level * bend, 0.0f));
        u32 mask = 0;
#pragma unroll
        for (u32 j = 0; j < kBinEdge; ++j) {
            const float y0 = yc + ((float)(j * LMK_GS_TILE) - h), y1 = yc + ((float)(j * LMK_GS_TILE) + h);
            const float yR = __builtin_amdgcn_fmed3f(yr, y0, y1), yL = __builtin_amdgcn_fmed3f(-yr, y0, y1);
            const float dR = (level - cn * yR * yR) * inv, dL = (level - cn * yL * yL) * inv;
            const float right = t.rx * yR + __builtin_amdgcn_sqrtf(fmaxf(dR, 0.0f)), left = t.rx * yL - __builtin_amdgcn_sqrtf(fmaxf(dL, 0.0f));
            const float hi = floorf(right / TS + hi0), lo = ceilf(left / TS + lo0);
            const u32 c1 = (u32)__builtin_amdgcn_fmed3f(hi, 0.0f, (float)kBinEdge), c0 = (u32)__builtin_amdgcn_fmed3f(lo, 0.0f, (float)kBinEdge);
            const bool some = dR >= 0.0f && c1 > c0;
            mask |= (some ? (1u << c1) - (1u << c0) : 0u) << (kBinEdge * j);
        }
        return mask;
    };
    const bool sound = t.A > 0.0f && cn > 0.0f && slack + inv + fabsf(bend) + fabsf(t.rx) + fabsf(t.tau) < 3.0e38f;
    const u32 outer = inside(t.tau + slack), inner = inside(t.tau - slack);
    sure = sound ? inner & outer : 0u;
    open = sound ? outer & ~inner : (1u << kBinTiles) - 1u;
}

// t / w and t % w for t < 2^22 (a tile grid has at most 2^22 tiles), 1 <= w <= 4096; inv_w = 1 / w
__device__ __forceinline__ void div_tiles(u32 t, u32 w, float inv_w, u32 &row, u32 &col)
{
    u32 q = (u32)((float)t * inv_w);            // within one of the quotient
    int r = (int)(t - q * w);
    if (r < 0) { q -= 1u; r += (int)w; }
    else if (r >= (int)w) { q += 1u; r -= (int)w; }
    row = q; col = (u32)r;
}

}  // namespace lmk
#endif
