// Host build of the split of the primitives over the counting workgroups (lmk_gs_internal.h): every primitive belongs to one
// workgroup, and a walk of a share ends, up to the largest number of primitives that an argument can hold.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <initializer_list>

#include "lmk_gs_internal.h"

using namespace lmk;

int main()
{
    int bad = 0;
    const u32 sizes[] = { 1u, 511u, 512u, 513u, 65536u, 65537u, 131073u, 262145u, 2000000u, 5000001u, 0x7fffffffu, 0xffffff00u - 8192u, 0xfffff7ffu,
                          0xfffff800u, 0xfffff801u, 0xffffff00u, 0xffffffffu };
    for (u32 n : sizes)
        for (u32 tiles : { 16u, 8160u, 8161u, 32768u, 32769u })
            for (int ordered = 0; ordered < 2; ++ordered) {
                const u32 block = bin_block(n, tiles, ordered != 0);
                bad += block > 2048u && ordered;
                const u32 groups = scratch_layout(n, 0, tiles).bin_blocks;
                u64 next = 0;
                for (u32 b = 0; b < groups; ++b) {
                    const BinShare s = bin_share(b, block, n);
                    if (s.count == 0u) { bad += next != n; continue; }
                    bad += s.beg != next || s.count > block || (u64)s.beg + s.count > n;
                    u32 rounds = 0;
                    for (u32 first = 0; first < s.count && rounds < 100; first += 2048u) ++rounds;
                    bad += rounds != (s.count + 2047u) / 2048u;
                    next = (u64)s.beg + s.count;
                }
                bad += next != n;
            }
    printf("bin share driver %s: %d\n", bad ? "FAILED" : "done", bad);
    return bad ? 1 : 0;
}
