// Cross-lane operations shared by the encode and decode kernels.
#pragma once
#include "csr_internal.h"

namespace csr {
namespace lane {

// Cross-lane reductions without the LDS: data-parallel-primitive moves
// inside a row of 16 lanes, lane reads across the four rows.  The order of the operations is fixed.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_mov(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v) { return __uint_as_float(dpp_mov<CTRL>(__float_as_uint(v))); }
template <int CTRL> __device__ __forceinline__ unsigned long long dpp_mov(unsigned long long v)
{
    return ((unsigned long long)dpp_mov<CTRL>((uint32_t)(v >> 32)) << 32) | dpp_mov<CTRL>((uint32_t)v);
}
// every lane gets op over its group of LANES (4, 8 or 16) neighbouring lanes
template <int LANES, typename T, typename Op> __device__ __forceinline__ T row_reduce(T v, Op op)
{
    v = op(v, dpp_mov<0xB1>(v));                            // quad_perm [1,0,3,2]
    v = op(v, dpp_mov<0x4E>(v));                            // quad_perm [2,3,0,1]
    if constexpr (LANES >= 8) v = op(v, dpp_mov<0x141>(v));  // row_half_mirror: the other quad of every 8
    if constexpr (LANES >= 16) v = op(v, dpp_mov<0x140>(v)); // row_mirror: the other half of the row
    return v;
}
__device__ __forceinline__ uint32_t lane_read(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }
__device__ __forceinline__ float lane_read(float v, int l) { return __uint_as_float(lane_read(__float_as_uint(v), l)); }
__device__ __forceinline__ unsigned long long lane_read(unsigned long long v, int l)
{
    return ((unsigned long long)lane_read((uint32_t)(v >> 32), l) << 32) | lane_read((uint32_t)v, l);
}
template <typename T, typename Op> __device__ __forceinline__ T wave_reduce(T v, Op op)
{
    v = row_reduce<16>(v, op);
    return op(op(lane_read(v, 0), lane_read(v, 16)), op(lane_read(v, 32), lane_read(v, 48)));
}
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct OpAdd { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; } };
struct OpMaxU { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };
struct OpOr { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a | b; } };
__device__ __forceinline__ float wave_max(float v) { return wave_reduce(v, OpMax()); }
__device__ __forceinline__ float wave_sum(float v) { return wave_reduce(v, OpAdd()); }

}  // namespace lane
}  // namespace csr
