// Cross-lane helpers shared by the kernels (64-lane wavefronts): a lane reads a register of
// another lane through ds_bpermute (no LDS memory involved), and a value every lane holds
// identically is moved to scalar registers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ntp {

__device__ __forceinline__ int bperm_i(int src_lane, int v) {
    return __builtin_amdgcn_ds_bpermute(src_lane << 2, v);
}
__device__ __forceinline__ float bperm_f(int src_lane, float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src_lane << 2, __float_as_int(v)));
}
// Sum / maximum over the groups of L consecutive lanes (every lane gets it): the xor tree 1, 2, 4, ...  Inside a row of 16
// lanes the partner's value comes through a DPP operand of the add itself (quad permutes, then mirrors: after the
// steps below, all lanes of a quad or half row hold the same value, so a mirrored lane is as good as the xor partner);
// wider steps go through the cross-lane network.
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int L> __device__ __forceinline__ float group_sum(float v, int lane) {
    if constexpr (L > 1) v += dpp_f<0xB1>(v);          // quad_perm [1,0,3,2]
    if constexpr (L > 2) v += dpp_f<0x4E>(v);          // quad_perm [2,3,0,1]
    if constexpr (L > 4) v += dpp_f<0x141>(v);         // row_half_mirror
    if constexpr (L > 8) v += dpp_f<0x140>(v);         // row_mirror
#pragma unroll
    for (int off = 16; off < L; off <<= 1) v += bperm_f(lane ^ off, v);
    return v;
}
template <int L> __device__ __forceinline__ float group_max(float v, int lane) {
    if constexpr (L > 1) v = fmaxf(v, dpp_f<0xB1>(v));
    if constexpr (L > 2) v = fmaxf(v, dpp_f<0x4E>(v));
    if constexpr (L > 4) v = fmaxf(v, dpp_f<0x141>(v));
    if constexpr (L > 8) v = fmaxf(v, dpp_f<0x140>(v));
#pragma unroll
    for (int off = 16; off < L; off <<= 1) v = fmaxf(v, bperm_f(lane ^ off, v));
    return v;
}
// lane j's value of every group of L lanes (j a constant)
template <int L, int J> __device__ __forceinline__ int group_bcast(int v, int lane) {
    if constexpr (L == 16) return __builtin_amdgcn_update_dpp(0, v, 0x150 + J, 0xf, 0xf, true);      // row_newbcast
    else return bperm_i((lane & ~(L - 1)) + J, v);
}
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v & 0xffffffff));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The group of an AggArgs that wavefront `wave` belongs to.  One entry after the other: most wavefronts are in the first ones (28,343
// vertices of 7 entries F = 64 9.45 us where the whole table is compared, 9.35 so; 100,000 of 5 F = 32 13.4 / 13.1).
template <class Args> __device__ __forceinline__ int agg_group_of(const Args& a, int wave) {
    int g = 0;
    while (g + 1 < (int)(sizeof a.wave_start / sizeof a.wave_start[0]) && wave >= a.wave_start[g + 1]) ++g;
    return g;
}

}  // namespace ntp
