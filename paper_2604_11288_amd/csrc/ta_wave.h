// Cross-lane reductions and scans of a 64-lane wavefront on the data-parallel-primitive path (no LDS
// round trips).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ta {

// ---- reductions: neighbours within quads, quads within a row of 16 by rotation, then the last lane of a row
// broadcast to the next row(s); lane 63 ends up with the reduction over the wavefront
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
#define TA_DPP_STEPS(STEP) STEP(0xb1) STEP(0x4e) STEP(0x124) STEP(0x128) STEP(0x142) STEP(0x143)

__device__ __forceinline__ float wave_max_dpp(float v)
{
#define STEP(C) v = fmaxf(v, __int_as_float(dpp_move<C>(__float_as_int(v))));
    TA_DPP_STEPS(STEP)
#undef STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_sum_dpp(float v)
{
#define STEP(C) v += __int_as_float(dpp_move<C>(__float_as_int(v)));
    TA_DPP_STEPS(STEP)
#undef STEP
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ int wave_min_dpp(int v)
{
#define STEP(C) { const int o = dpp_move<C>(v); v = o < v ? o : v; }
    TA_DPP_STEPS(STEP)
#undef STEP
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ uint32_t wave_min_dpp(uint32_t v)
{
#define STEP(C) { const uint32_t o = (uint32_t)dpp_move<C>((int)v); v = o < v ? o : v; }
    TA_DPP_STEPS(STEP)
#undef STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_max_dpp(uint32_t v)
{
#define STEP(C) { const uint32_t o = (uint32_t)dpp_move<C>((int)v); v = o > v ? o : v; }
    TA_DPP_STEPS(STEP)
#undef STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned long long wave_min_dpp(unsigned long long v)
{
#define STEP(C) { const unsigned lo = (unsigned)dpp_move<C>((int)(unsigned)v), hi = (unsigned)dpp_move<C>((int)(unsigned)(v >> 32)); \
                  const unsigned long long o = ((unsigned long long)hi << 32) | lo; v = o < v ? o : v; }
    TA_DPP_STEPS(STEP)
#undef STEP
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
    return ((unsigned long long)hi << 32) | lo;
}
#undef TA_DPP_STEPS

// ---- inclusive sum over the lanes up to this one
__device__ __forceinline__ uint32_t wave_scan_dpp(uint32_t v)
{
#define STEP(CTRL, ROWS) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
    STEP(0x111, 0xf) STEP(0x112, 0xf) STEP(0x114, 0xf) STEP(0x118, 0xf)   // shifts right by 1, 2, 4, 8 within rows of 16
    STEP(0x142, 0xa) STEP(0x143, 0xc)                                     // last lane of a row to the next; lane 31 to the upper half
#undef STEP
    return v;
}
// sum over the wavefront (integers: exact in any order)
__device__ __forceinline__ uint32_t wave_sum_dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_dpp(v), 63);
}
__device__ __forceinline__ int wave_sum_dpp(int v) { return (int)wave_sum_dpp((uint32_t)v); }

}  // namespace ta
