// Rows of at most 128 elements held by a group of SUB = 8, 16 or 32 lanes, 64 / SUB of them side by side in a wave: lane
// sl of a group owns elements 4*sl .. 4*sl+3.
#pragma once
#include "dev_common.h"

// sum over the lanes of a group, the same bits in all of them: in-row moves, and for 32 lanes one swap of rows
template <int SUB>
__device__ __forceinline__ float group_sum(float x)
{
    static_assert(SUB == 8 || SUB == 16 || SUB == 32, "group sizes");
    x += dpp_get<0xB1, 0xF>(x);                  // quad_perm [1,0,3,2]
    x += dpp_get<0x4E, 0xF>(x);                  // quad_perm [2,3,0,1]
    x += dpp_get<0x141, 0xF>(x);                 // row_half_mirror
    if (SUB >= 16) x += dpp_get<0x140, 0xF>(x);  // row_mirror
    if (SUB == 32) x += __shfl_xor(x, 16, WAVE);
    return x;
}
// sum over the groups of a wave, lane by lane
template <int SUB>
__device__ __forceinline__ float4 sum_groups(float4 v)
{
#pragma unroll
    for (int o = SUB; o < WAVE; o <<= 1) {
        v.x += __shfl_xor(v.x, o, WAVE);
        v.y += __shfl_xor(v.y, o, WAVE);
        v.z += __shfl_xor(v.z, o, WAVE);
        v.w += __shfl_xor(v.w, o, WAVE);
    }
    return v;
}
__device__ __forceinline__ float dot4(float4 a, float4 b) { return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x))); }
__device__ __forceinline__ void axpy4(float4 &acc, float a, float4 x)
{
    acc.x = fmaf(a, x.x, acc.x);
    acc.y = fmaf(a, x.y, acc.y);
    acc.z = fmaf(a, x.z, acc.z);
    acc.w = fmaf(a, x.w, acc.w);
}
static inline int group_lanes(int D) { return D > 64 ? 32 : D > 32 ? 16 : 8; }
