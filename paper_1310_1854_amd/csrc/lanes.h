// lanes.h -- exchanges between the lanes of a wave: broadcasts of one lane's
// value and data-parallel-primitive (DPP) moves, which need no LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vrt {

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

__device__ __forceinline__ double lane_f64(double v, int l)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint64_t r = (uint64_t)lane_u32((uint32_t)u, l) | ((uint64_t)lane_u32((uint32_t)(u >> 32), l) << 32);
    return __longlong_as_double((long long)r);
}

// DPP moves; lanes without a source keep their own value.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint64_t r = (uint64_t)dpp_u32<CTRL>((uint32_t)u) | ((uint64_t)dpp_u32<CTRL>((uint32_t)(u >> 32)) << 32);
    return __longlong_as_double((long long)r);
}

// Minimum and maximum over the wave (row shifts, then row broadcasts; the
// result is lane 63's).
#define VRT_WAVE_REDUCE(v, op, dpp)  \
    v = op(v, dpp<0x111>(v));        \
    v = op(v, dpp<0x112>(v));        \
    v = op(v, dpp<0x114>(v));        \
    v = op(v, dpp<0x118>(v));        \
    v = op(v, dpp<0x142>(v));        \
    v = op(v, dpp<0x143>(v))
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    VRT_WAVE_REDUCE(v, min, dpp_u32);
    return lane_u32(v, 63);
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    VRT_WAVE_REDUCE(v, max, dpp_u32);
    return lane_u32(v, 63);
}
__device__ __forceinline__ double wave_min_f64(double v)
{
    VRT_WAVE_REDUCE(v, fmin, dpp_f64);
    return lane_f64(v, 63);
}
__device__ __forceinline__ double wave_max_f64(double v)
{
    VRT_WAVE_REDUCE(v, fmax, dpp_f64);
    return lane_f64(v, 63);
}

// Exchanges between the halves of a group of 8 or 16 lanes whose halves
// already agree: quad permutes, then the mirrors of 8 and 16 lanes. F gets
// the move as an object and combines the lane's values with the other
// half's. Every lane of these moves has a source, so they may be folded into
// the instruction that uses them.
template <int CTRL>
struct Swap {
    static __device__ __forceinline__ uint32_t u32(uint32_t v)
    {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
    }
    static __device__ __forceinline__ int32_t i32(int32_t v) { return (int32_t)u32((uint32_t)v); }
    static __device__ __forceinline__ float f32(float v) { return __uint_as_float(u32(__float_as_uint(v))); }
    static __device__ __forceinline__ double f64(double v)
    {
        const uint64_t u = (uint64_t)__double_as_longlong(v);
        return __longlong_as_double((long long)((uint64_t)u32((uint32_t)u) | ((uint64_t)u32((uint32_t)(u >> 32)) << 32)));
    }
};
template <int W, class F>
__device__ __forceinline__ void group_exchange(F &&f)
{
    static_assert(W == 8 || W == 16, "groups of half a row or a row");
    f(Swap<0xB1>());    // quad_perm 1 0 3 2
    f(Swap<0x4E>());    // quad_perm 2 3 0 1
    f(Swap<0x141>());   // row_half_mirror
    if (W == 16) f(Swap<0x140>());   // row_mirror
}

// The bits of a ballot that belong to this lane's group.
template <int W>
__device__ __forceinline__ uint32_t group_bits(uint64_t ballot)
{
    return (uint32_t)(ballot >> (threadIdx.x & 63 & ~(W - 1))) & ((1u << W) - 1u);
}

}  // namespace vrt
