// Wavefront sums and broadcasts of doubles for the one-wavefront-per-object
// quadric kernels, whose time is the latency of one dependent FP64 chain.
#pragma once
#include "dqo_device.hpp"

namespace dqo {

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// The value of lane ^ D: DPP moves inside a row of 16 lanes (a ds_bpermute per
// word, as __shfl_xor compiles to, costs an LDS round trip each).
template <int D>
__device__ __forceinline__ double lane_xor(double x) {
    if constexpr (D == 1) return dpp_f64<0xB1>(x);   // quad_perm [1,0,3,2]
    if constexpr (D == 2) return dpp_f64<0x4E>(x);   // quad_perm [2,3,0,1]
    if constexpr (D == 4) {                          // even banks of 4 lanes take lane + 4, odd ones lane - 4
        int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x104, 0xF, 0x5, false);
        int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x104, 0xF, 0x5, false);
        lo = __builtin_amdgcn_update_dpp(lo, __double2loint(x), 0x114, 0xF, 0xA, false);
        hi = __builtin_amdgcn_update_dpp(hi, __double2hiint(x), 0x114, 0xF, 0xA, false);
        return __hiloint2double(hi, lo);
    }
    if constexpr (D == 8) return dpp_f64<0x128>(x);  // row_ror:8
    return __shfl_xor(x, D);
}
// x of lane l plus x of lane l ^ 32 (l ^ 16): a half-wave (row) swap of the
// value with itself leaves the two addends in the two results.
__device__ __forceinline__ double add_xor32(double x) {
    const uint32_t lo = (uint32_t)__double2loint(x), hi = (uint32_t)__double2hiint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}
__device__ __forceinline__ double add_xor16(double x) {
    const uint32_t lo = (uint32_t)__double2loint(x), hi = (uint32_t)__double2hiint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}
// Sum over the wavefront in every lane, as the butterfly over lane distances
// 32, 16, 8, 4, 2, 1 (a + b == b + a exactly: every lane ends equal).
__device__ __forceinline__ double wave_sum_all(double v) {
    v = add_xor32(v);
    v = add_xor16(v);
    v += lane_xor<8>(v);
    v += lane_xor<4>(v);
    v += lane_xor<2>(v);
    v += lane_xor<1>(v);
    return v;
}
// The value of one lane (uniform index) in every lane, through scalar registers.
__device__ __forceinline__ double lane_value(double x, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

}  // namespace dqo
