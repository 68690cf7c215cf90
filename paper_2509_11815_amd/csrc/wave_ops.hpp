// Cross-lane reductions of a wavefront on the vector ALU (DPP), a few cycles per step; the shuffle
// intrinsics go through the LDS crossbar, ten times as long per step.
#pragma once
#include "common.hpp"

namespace specvlm {

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int dpp(int x) { return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false); }

constexpr int kRor1 = 0x121, kRor2 = 0x122, kRor4 = 0x124, kRor8 = 0x128;     // rotate a row of 16 lanes

// Over each row of 16 lanes; every lane of the row gets the result.
__device__ __forceinline__ float row_max(float x) {
    x = fmaxf(x, dpp<kRor8>(x));
    x = fmaxf(x, dpp<kRor4>(x));
    x = fmaxf(x, dpp<kRor2>(x));
    return fmaxf(x, dpp<kRor1>(x));
}
template <typename T>
__device__ __forceinline__ T row_sum(T x) {
    x += dpp<kRor8>(x);
    x += dpp<kRor4>(x);
    x += dpp<kRor2>(x);
    return x + dpp<kRor1>(x);
}

__device__ __forceinline__ float lane_of(float x, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane)); }

// Over the wavefront; uniform result.
__device__ __forceinline__ float wave_max(float x) {
    x = row_max(x);
    return fmaxf(fmaxf(lane_of(x, 0), lane_of(x, 16)), fmaxf(lane_of(x, 32), lane_of(x, 48)));
}
__device__ __forceinline__ float wave_sum(float x) {
    x = row_sum(x);
    return (lane_of(x, 0) + lane_of(x, 16)) + (lane_of(x, 32) + lane_of(x, 48));
}

}  // namespace specvlm
