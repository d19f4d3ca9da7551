// Device helpers shared by the strip kernels: wave shifts and sums with DPP
// moves, and the refined division of the smoothers.
#pragma once

#include <hip/hip_runtime.h>

namespace mbp {

// Sum over the 64 lanes of a wave with DPP moves (no LDS round trips);
// lane 63 ends up with the total.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// a / d by a hardware reciprocal refined with Newton-Raphson steps and one
// residual correction of the quotient (d is a nonzero diagonal of moderate
// magnitude here).  Of 4 million random quotients in each precision every one was
// the rounded one, as IEEE division gives it.
__device__ __forceinline__ double div_nr(double a, double d) {
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    const double q = a * r;
    return fma(fma(-d, q, a), r, q);
}
__device__ __forceinline__ float div_nr(float a, float d) {
    float r = __builtin_amdgcn_rcpf(d);
    r = fmaf(r, fmaf(-d, r, 1.0f), r);
    const float q = a * r;
    return fmaf(fmaf(-d, q, a), r, q);
}

__device__ __forceinline__ double wave_sum63(double v) {
    v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]: every lane holds its quad's sum
    v += dpp_move<0x114>(v);  // row_shr:4
    v += dpp_move<0x118>(v);  // row_shr:8: lane 15 of each row holds the row's sum
    v += dpp_move<0x142>(v);  // row_bcast:15
    v += dpp_move<0x143>(v);  // row_bcast:31
    return v;
}

// value of lane - 1 (0 at lane 0) and of lane + 1 (0 at lane 63)
template <int CTRL>
__device__ __forceinline__ double dpp_shift(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ float dpp_shift(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <typename T>
__device__ __forceinline__ T from_left(T v) { return dpp_shift<0x138>(v); }
template <typename T>
__device__ __forceinline__ T from_right(T v) { return dpp_shift<0x130>(v); }

}  // namespace mbp
