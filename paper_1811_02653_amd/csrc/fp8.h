// fp8.h -- OCP E4M3 encoding with E8M0 block scales, shared by the
// quantization kernels and the sketch kernel's quantizing epilogue.
//
// Per block of 64 values: s = the smallest integer with max|x| <= 448 * 2^s
// (so nothing saturates), clamped to [-127, 127]; code = RNE(x * 2^-s) in
// E4M3 (4 exponent bits, bias 7, 3 fraction bits; largest finite value 448,
// subnormals down to 2^-9).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace osk {

// s of a block whose largest |x| has these FP32 bits.  (amax = f * 2^E, f in
// [0.5, 1): 448 = 0.875 * 2^9, so amax <= 448 * 2^s from s = E - 9 when f <=
// 0.875, else E - 8.  A subnormal amax lands below the clamp either way.)  The
// bits order like the values, with infinities and NaN above every finite one.
__device__ __forceinline__ int e8m0_exponent(uint32_t amax) {
    const int s = (int)(amax >> 23) - 126 - 9 + ((amax & 0x7FFFFFu) > 0x600000u ? 1 : 0);
    return max(-127, s);
}

// E4M3 codes of four values |v| <= 448, v0 in the low byte (hardware
// conversion, round to nearest even; an infinity or NaN becomes the E4M3 NaN).
__device__ __forceinline__ uint32_t e4m3_pack4(float v0, float v1, float v2, float v3) {
    const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(v0, v1, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v2, v3, lo, true);
}

__device__ __forceinline__ uint32_t abs_bits(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

// max(x, x of another lane picked by the DPP control), 0 where that lane is
// outside the row
template <int kCtrl, int kRows = 0xF>
__device__ __forceinline__ uint32_t dpp_max(uint32_t x) {
    return max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRows, 0xF, true));
}

__device__ __forceinline__ float e4m3_value(uint32_t code) {
    const uint32_t e = (code >> 3) & 0xFu, m = code & 7u;
    const float mag = e ? ldexpf(1.f + (float)m * 0.125f, (int)e - 7) : (float)m * 0.001953125f;
    return (code & 0x80u) ? -mag : mag;
}

}  // namespace osk
