// Host build of the library's device headers, for properties that need millions of random inputs: which 4x4 cells an entry is
// listed in (blend_reach.h), how many tiles of a row are kept (tile_test.h), which workgroup takes which tile
// (tile_work.h).  Prints what it counted; anything but 0 as exit code is a failure.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <algorithm>
#include <random>
#include <vector>

#include "blend_reach.h"
#include "tile_test.h"
#include "tile_work.h"

using namespace lmk;

static std::mt19937_64 rng(1);
static double uniform(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }
static uint64_t below(uint64_t n) { return std::uniform_int_distribution<uint64_t>(0, n - 1)(rng); }
static const float kInf = INFINITY;

struct Conic { float A, B, C; double a, c; };
// the inverse of a 2D covariance in fp32, as the projection computes it: round ones, ellipses, needles; axes up to `most` pixels
static bool draw_conic(double most, Conic &k)
{
    const double l1 = exp(uniform(log(0.3), log(most))), l2 = below(3) ? exp(uniform(log(0.3), log(l1 < 0.4 ? 0.4 : l1))) : 0.3;
    const double th = below(4) ? uniform(0.0, M_PI) : (double)below(4) * M_PI / 4.0 + (below(2) ? 0.0 : uniform(-1e-3, 1e-3));
    const double s = sin(th), co = cos(th);
    const float a = (float)(l1 * l1 * co * co + l2 * l2 * s * s), b = (float)((l1 * l1 - l2 * l2) * s * co),
                c = (float)(l1 * l1 * s * s + l2 * l2 * co * co);
    const float ac = a * c, bb = b * b, det = ac - bb;
    if (!(det > 0.0f)) return false;
    k = { c / det, -b / det, a / det, a, c };
    return true;
}

static u32 listed_cells(const StagedEntry &e, const float4 *record)
{
    const u32 mask = entry_cells(e);
    return mask == kNoEllipse ? entry_cells_any(e, record, 0u) : mask;
}

static int cells(uint64_t count)
{
    uint64_t listed = 0, vain = 0, missed = 0, tested = 0;
    while (tested < count) {
        Conic k;
        if (!draw_conic(tested % 5 ? 60.0 : 3000.0, k)) continue;
        const float o = tested % 4 ? (float)uniform(1.0 / 255.0, 1.0) : (float)((1.0 + uniform(0.0, 1e-4)) / 255.0);
        // centres where the level reaches the tile's surroundings, seen from its reference point
        const double wide = 12.0 + 3.5 * sqrt(k.a), high = 12.0 + 3.5 * sqrt(k.c);
        const float4 fa = make_float4((float)uniform(-wide, wide), (float)uniform(-high, high), k.A, k.B), fb = make_float4(k.C, o, 0.f, 0.f);
        const StagedEntry e = stage_entry(fa, fb, 0.0f, 0.0f, 0.0f);
        float4 record[3] = { fa, fb, make_float4(0.f, 0.f, 0.f, 0.f) };
        const u32 mask = listed_cells(e, record);
        u32 reached = 0;
        for (int j = 0; j < 16; ++j)
            for (int i = 0; i < 16; ++i) {
                const float l = log2_alpha(e.geo, e.cop, e.geo.x - ((float)i - 3.5f), e.geo.y - ((float)j - 3.5f));
                if (!(exp2f(l) < 1.0f / 255.0f)) reached |= 1u << (4 * (j / 4) + i / 4);
            }
        missed += __builtin_popcount(reached & ~mask);
        listed += __builtin_popcount(mask);
        vain += __builtin_popcount(mask & ~reached);
        ++tested;
    }
    printf("cells: %llu entries, %llu cells listed, %llu of them reach no pixel, %llu missed\n", (unsigned long long)tested,
           (unsigned long long)listed, (unsigned long long)vain, (unsigned long long)missed);
    return missed != 0 || vain * 20 > listed;
}

// entries whose conic holds a NaN, or an infinity on its diagonal, are listed nowhere; a singular conic is listed where it reaches
static int odd_cells()
{
    int bad = 0;
    for (int comp = 0; comp < 3; ++comp)
        for (float value : { (float)NAN, kInf })
            for (int k = 0; k < 1000; ++k) {
                if (comp == 1 && value == kInf) continue;
                float f[3] = { (float)uniform(0.01, 1.0), (float)uniform(-0.005, 0.005), (float)uniform(0.01, 1.0) };
                f[comp] = value;
                const float4 record[2] = { make_float4((float)uniform(-20, 20), (float)uniform(-20, 20), f[0], f[1]), make_float4(f[2], 0.9f, 0.f, 0.f) };
                bad += listed_cells(stage_entry(record[0], record[1], 0.0f, 0.0f, 0.0f), record) != 0u;
            }
    const float4 line[2] = { make_float4(4.0f, 4.0f, 1.0f, 1.0f), make_float4(1.0f, 0.9f, 0.f, 0.f) };       // along x + y = const
    const u32 diagonal = listed_cells(stage_entry(line[0], line[1], 0.0f, 0.0f, 0.0f), line);
    bad += (diagonal & 0x1248u) == 0u || (diagonal & 0x8000u) != 0u;
    printf("odd cells: %d wrong, diagonal %04x\n", bad, diagonal);
    return bad;
}

// rows of random ellipses at thresholds of all opacities; with `odd`, at thresholds around and below zero, and of values that are no
// ellipse (NaN, infinities, the largest numbers in each field, conics of no or negative determinant)
static int rows(uint64_t count, bool odd)
{
    uint64_t tested = 0, differ = 0, kept = 0;
    while (tested < count) {
        Conic k;
        const double most = tested % 7 ? 600.0 : 1e5;
        if (!draw_conic(most, k)) continue;
        const float tau = (float)(odd ? uniform(-0.01, 0.02) : uniform(0.01, 11.1));
        const u32 x0 = (u32)below(40), x1 = x0 + 1u + (u32)below(250), y0 = (u32)below(40), y1 = y0 + 1u + (u32)below(60);
        const double hx = sqrt(11.09 * k.a), hy = sqrt(11.09 * k.c);
        TileTest t = make_tile_test((float)uniform(16.0 * x0 - hx, 16.0 * x1 + hx), (float)uniform(16.0 * y0 - hy, 16.0 * y1 + hy), k.A, k.B, k.C, tau);
        if (odd && below(3)) {
            const float values[6] = { NAN, kInf, -kInf, 3e38f, -3e38f, 0.0f };
            if (below(2)) {
                float *const field[6] = { &t.u, &t.v, &t.A, &t.B, &t.C, &t.tau };
                for (u32 m = (u32)below(2); m < 2; ++m) *field[below(6)] = values[below(6)];
                t = make_tile_test(t.u, t.v, t.A, t.B, t.C, t.tau);
            } else {
                const float B = (float)(sqrt((double)k.A * k.C) * uniform(0.999999, 1.5)) * (below(2) ? 1.0f : -1.0f);
                t = make_tile_test(t.u, t.v, k.A, B, k.C, (float)uniform(0.01, 11.1));
            }
        }
        const float fx = fmaxf(fabsf((float)(x0 * LMK_GS_TILE) - t.u), fabsf((float)(x1 * LMK_GS_TILE) - t.u));
        const float fy = fmaxf(fabsf((float)(y0 * LMK_GS_TILE) - t.v), fabsf((float)(y1 * LMK_GS_TILE) - t.v));
        const float slack = 2e-5f * (t.A * fx * fx + t.C * fy * fy);
        for (u32 n = 0; n < 8; ++n) {
            const u32 ty = y0 + (u32)below(y1 - y0);
            u32 want = 0;
            for (u32 tx = x0; tx < x1; ++tx) want += tile_kept(t, tx, ty) ? 1u : 0u;
            differ += row_kept(t, ty, x0, x1, slack) != want;
            kept += want;
            ++tested;
        }
    }
    printf("%srows: %llu, %llu tiles kept, %llu rows differ\n", odd ? "odd " : "", (unsigned long long)tested, (unsigned long long)kept, (unsigned long long)differ);
    return differ != 0;
}

// every tile whole by one workgroup, or its four shares by one each, these on one die; shared are exactly the long lists
static int work(u32 tiles, int kind, bool ordered, bool all_bad, u32 most)
{
    std::vector<u64> len(tiles), offsets(tiles + 1, 0);
    for (u32 t = 0; t < tiles; ++t) {
        const double u = uniform(1e-6, 1.0);
        len[t] = kind == 0 ? below(2000) : kind == 1 ? (u64)(10.0 / u) : kind == 2 ? 0u : kind == 3 ? (t % 97 == 5 ? 5000u : below(60)) : 700u;
        offsets[t + 1] = offsets[t] + len[t];
    }
    std::vector<u32> order(tiles);
    for (u32 t = 0; t < tiles; ++t) order[t] = t;
    std::shuffle(order.begin(), order.end(), rng);
    // as the tile scan orders them: by power of two, those that may be shared first
    auto bucket = [&](u32 t) { return 2 * (len[t] > 1 ? 64 - __builtin_clzll(len[t] - 1) : 0) + (len[t] >= long_list_from(offsets[tiles]) ? 1 : 0); };
    std::stable_sort(order.begin(), order.end(), [&](u32 x, u32 y) { return bucket(x) > bucket(y); });
    if (all_bad) for (u32 &t : order) t = 0xffffffffu - (u32)below(100);
    std::vector<u32> whole(tiles, 0), shares(tiles, 0), die(tiles, 8);
    int bad = 0, shared = 0;
    for (u32 b = 0; b < tile_work_grid(tiles, ordered); ++b) {
        const TileWork w = tile_work(b, tiles, ordered ? order.data() : nullptr, offsets.data(), most);
        if (w.whole > tiles || w.shared > tiles || w.share > 3u) { ++bad; continue; }
        if (w.whole < tiles) ++whole[w.whole];
        if (w.shared < tiles) {
            bad += (shares[w.shared] >> w.share) & 1u;
            shares[w.shared] |= 1u << w.share;
            if (die[w.shared] == 8) die[w.shared] = b % 8;
            bad += die[w.shared] != b % 8;
        }
    }
    u32 longs = 0;
    for (u32 t = 0; t < tiles; ++t) longs += len[t] >= long_list_from(offsets[tiles]) ? 1u : 0u;
    const bool by_length = ordered && !all_bad && tiles > kSharedTiles && tiles <= kSharedMaxTiles && offsets[tiles] != 0u;
    for (u32 t = 0; t < tiles; ++t) {
        const bool one = (whole[t] == 1 && shares[t] == 0) || (whole[t] == 0 && shares[t] == 15);
        bad += all_bad && ordered ? (whole[t] || shares[t]) : !one;
        if (by_length) bad += (shares[t] == 15) != (longs <= most && len[t] >= long_list_from(offsets[tiles]));
        shared += shares[t] == 15;
    }
    if (bad) printf("work: %u tiles, lists %d, ordered %d: %d wrong, %d shared\n", tiles, kind, (int)ordered, bad, shared);
    return bad ? 1 : 0;
}

int main()
{
    int bad = cells(1000000) + odd_cells() + rows(500000, false) + rows(500000, true);
    int runs = 0;
    for (u32 tiles : { 1u, 6u, 7u, 8u, 9u, 255u, 256u, 257u, 258u, 271u, 272u, 273u, 294u, 306u, 383u, 384u, 385u, 475u, 608u, 760u, 767u, 768u,
                       769u, 770u, 783u, 1200u, 1900u, 2047u, 2048u, 2049u, 8160u })
        for (int kind = 0; kind < 5; ++kind)
            for (int ordered = 0; ordered < 2; ++ordered)
                for (int all_bad = 0; all_bad < 2; ++all_bad)
                    for (u32 most : { 128u, 256u }) { ++runs; bad += work(tiles, kind, ordered != 0, all_bad != 0, most); }
    printf("work: %d grids\nheaders driver %s\n", runs, bad ? "FAILED" : "done");
    return bad ? 1 : 0;
}
