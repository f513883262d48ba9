// What the library's device headers need of a compiler for the GPU, for a host build of them by g++ in the tests: plain
// arithmetic in place of the instructions.  The reciprocal and the square root are the GPU's to one ulp only, so they come with
// a random error of that size here.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>

#define __device__
#define __host__
#define __forceinline__ inline

struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
static inline float4 make_float4(float x, float y, float z, float w) { return { x, y, z, w }; }
typedef struct { int unused; } *hipStream_t;
typedef int hipError_t;

static uint64_t noise_state = 88172645463325252ull;
static inline float noisy(float x)
{
    noise_state ^= noise_state << 13; noise_state ^= noise_state >> 7; noise_state ^= noise_state << 17;
    return x * (1.0f + 1.1920929e-7f * (float)((int)(noise_state % 3u) - 1));
}
#define __log2f(x) noisy(log2f(x))
static inline uint32_t __float_as_uint(float x) { uint32_t u; memcpy(&u, &x, 4); return u; }
static inline float __int_as_float(int i) { float x; memcpy(&x, &i, 4); return x; }
static inline int __float_as_int(float x) { int i; memcpy(&i, &x, 4); return i; }
static inline float __builtin_amdgcn_rcpf(float x) { return noisy(1.0f / x); }
static inline float __builtin_amdgcn_sqrtf(float x) { return noisy(sqrtf(x)); }
static inline float __builtin_amdgcn_fmed3f(float a, float b, float c)
{
    return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c));
}
// across lanes: named by code that these tests do not run
static inline uint64_t __builtin_amdgcn_ballot_w64(bool) { return 0; }
static inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t, uint32_t) { return 0; }
static inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t, uint32_t) { return 0; }
static inline int __builtin_amdgcn_update_dpp(int, int, int, int, int, bool) { return 0; }
#define __builtin_amdgcn_fence(order, scope) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_sched_barrier(mask) ((void)0)
