// Host build of the test of a bin's tiles (tile_test.h): what it calls sure is kept, what it leaves out is not, by asking every
// tile, for millions of random ellipses.  Prints what it counted; anything but 0 as exit code is a failure.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <random>

#include "tile_test.h"

using namespace lmk;

static std::mt19937_64 rng(2);
static double uniform(double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); }
static uint64_t below(uint64_t n) { return std::uniform_int_distribution<uint64_t>(0, n - 1)(rng); }

int main()
{
    uint64_t tested = 0, tiles = 0, asked = 0, wrong = 0, odd = 0;
    while (tested < 3000000) {
        // round ones, ellipses, needles; axes up to hundreds, thousands, 1e5 pixels
        const double most = tested % 3 == 0 ? 60.0 : (tested % 7 ? 600.0 : 1e5);
        const double l1 = exp(uniform(log(0.3), log(most))), l2 = below(3) ? exp(uniform(log(0.3), log(l1 < 0.4 ? 0.4 : l1))) : 0.3;
        const double th = below(4) ? uniform(0.0, M_PI) : (double)below(4) * M_PI / 4.0 + (below(2) ? 0.0 : uniform(-1e-3, 1e-3));
        const double s = sin(th), co = cos(th);
        const float a = (float)(l1 * l1 * co * co + l2 * l2 * s * s), b = (float)((l1 * l1 - l2 * l2) * s * co), c = (float)(l1 * l1 * s * s + l2 * l2 * co * co);
        const float ac = a * c, bb = b * b, det = ac - bb;
        if (!(det > 0.0f)) continue;
        const u32 bx = 4u * (u32)below(60), by = 4u * (u32)below(60);
        const double wide = 64.0 + 3.5 * sqrt((double)a), high = 64.0 + 3.5 * sqrt((double)c);
        TileTest t = make_tile_test((float)(16.0 * bx + 32.0 + uniform(-wide, wide)), (float)(16.0 * by + 32.0 + uniform(-high, high)), c / det, -b / det, a / det,
                                    (float)(tested % 5 ? uniform(0.01, 11.1) : uniform(0.0, 0.02)));
        if (tested % 1000 == 1) {                            // values that are no ellipse: all have to be asked
            float *const field[5] = { &t.A, &t.C, &t.rx, &t.tau, &t.u };
            *field[below(5)] = below(2) ? NAN : INFINITY;
            u32 sure, open;
            bin_tiles(t, bx, by, sure, open);
            for (u32 k = 0; k < kBinTiles; ++k) {
                const bool kept = tile_kept(t, bx + k % kBinEdge, by + k / kBinEdge);
                odd += ((sure >> k) & 1u) && !kept;
                odd += !(((sure | open) >> k) & 1u) && kept;
            }
            ++tested;
            continue;
        }
        u32 sure, open;
        bin_tiles(t, bx, by, sure, open);
        for (u32 k = 0; k < kBinTiles; ++k) {
            const bool kept = tile_kept(t, bx + k % kBinEdge, by + k / kBinEdge);
            wrong += ((sure >> k) & 1u) && !kept;
            wrong += !(((sure | open) >> k) & 1u) && kept;
            tiles += kept;
        }
        wrong += (sure & open) != 0u;
        asked += __builtin_popcount(open);
        ++tested;
    }
    printf("bins: %llu, %llu tiles kept, %llu asked, %llu wrong, %llu of no ellipse\n", (unsigned long long)tested, (unsigned long long)tiles,
           (unsigned long long)asked, (unsigned long long)wrong, (unsigned long long)odd);
    const bool bad = wrong != 0 || odd != 0 || asked * 4 > tiles;
    printf("bin tiles driver %s\n", bad ? "FAILED" : "done");
    return bad ? 1 : 0;
}
