// Sums, scans and extremes over a wavefront.
#ifndef LMK_GS_WAVE_OPS_H
#define LMK_GS_WAVE_OPS_H
#include "lmk_gs_internal.h"

namespace lmk {

// Over the 64 lanes, all of them active: inclusive sum and largest value so far; least and largest value and sum, the same in every lane.  Lane exchanges
// that need no LDS: shifts by 1, 2, 4, 8 inside the rows of 16, then the last lane of a row to the next row and of the first
// half to the second.
template <int CTRL, int ROWS>
__device__ __forceinline__ u32 wave_dpp(u32 none, u32 v)
{
    return (u32)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xf, false);
}
template <class Join>
__device__ __forceinline__ u32 wave_join(u32 none, u32 v, Join &&join)
{
    v = join(v, wave_dpp<0x111, 0xf>(none, v));
    v = join(v, wave_dpp<0x112, 0xf>(none, v));
    v = join(v, wave_dpp<0x114, 0xf>(none, v));
    v = join(v, wave_dpp<0x118, 0xf>(none, v));
    v = join(v, wave_dpp<0x142, 0xa>(none, v));
    return join(v, wave_dpp<0x143, 0xc>(none, v));
}
__device__ __forceinline__ u32 wave_last(u32 v) { return (u32)__builtin_amdgcn_readlane((int)v, (int)kWave - 1); }
__device__ __forceinline__ u32 wave_scan(u32 v) { return wave_join(0u, v, [](u32 a, u32 b) { return a + b; }); }
__device__ __forceinline__ u32 wave_sum(u32 v) { return wave_last(wave_scan(v)); }
__device__ __forceinline__ u32 wave_min(u32 v) { return wave_last(wave_join(~0u, v, [](u32 a, u32 b) { return a < b ? a : b; })); }
__device__ __forceinline__ u32 wave_scan_max(u32 v) { return wave_join(0u, v, [](u32 a, u32 b) { return a > b ? a : b; }); }
__device__ __forceinline__ u32 wave_max(u32 v) { return wave_last(wave_scan_max(v)); }

}  // namespace lmk
#endif
