// OCP MX FP4 (E2M1) element arithmetic shared by the MXFP4 kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gift {

// floor(log2(a)) of a finite a > 0 from its bits (subnormals included)
__device__ __forceinline__ int mx_floor_log2(float a) {
  const uint32_t b = __float_as_uint(a);
  const int e = (int)(b >> 23);
  if (e > 0) return e - 127;
  return -149 + (31 - __clz((int)(b & 0x7fffffu)));
}

// scale exponent k of a block (amax over the block, bad = a NaN or an
// infinity in it): 2^k with k = floor(log2 amax) - 2, at least -127
__device__ __forceinline__ int mx_scale_exp(float amax, int bad) {
  int k = -127;
  if (!bad && amax > 0.f) {
    k = mx_floor_log2(amax) - 2;
    k = k < -127 ? -127 : k;
  }
  return k;
}

// E2M1 codes (sign in bit 3) of four values scaled by 2^-k, element e in bits
// 4 e .. 4 e + 3: the hardware conversion rounds to the nearest of 0, 0.5, 1,
// 1.5, 2, 3, 4, 6 with ties to the even code, saturates and keeps the sign of
// zero (one instruction per pair, where comparisons against the seven
// midpoints are some 20 per element).  A bad block's codes are zero.
__device__ __forceinline__ uint32_t mx_encode4(float v0, float v1, float v2, float v3, int k, int bad) {
  uint32_t w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, ldexpf(v0, -k), ldexpf(v1, -k), 1.0f, 0);
  w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, ldexpf(v2, -k), ldexpf(v3, -k), 1.0f, 1);
  return bad ? 0u : w & 0xffffu;
}

// exact values of the codes in byte B of w, before their scale
template <int B>
__device__ __forceinline__ void mx_decode2(uint32_t w, float &a, float &b) {
  const auto v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, B);
  a = v[0];
  b = v[1];
}

// exact dequantized values of four codes (NaN in a bad block)
__device__ __forceinline__ void mx_decode4(uint32_t w, int k, int bad, float (&d)[4]) {
  mx_decode2<0>(w, d[0], d[1]);
  mx_decode2<1>(w, d[2], d[3]);
#pragma unroll
  for (int e = 0; e < 4; ++e) d[e] = bad ? __int_as_float(0x7fc00000) : ldexpf(d[e], k);
}

}  // namespace gift
