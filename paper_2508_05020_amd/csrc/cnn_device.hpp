// Device helpers shared by the 2D and 3D predictor kernels: BF16 rounding,
// the 16x16x16 BF16 MFMA and 4-element operand loads.
//
// MFMA used: v_mfma_f32_16x16x16_bf16 (__builtin_amdgcn_mfma_f32_16x16x16bf16_1k).
// Operand layout per lane l (0..63), element e (0..3):
//   A[i][k]: i = l % 16, k = 4 (l / 16) + e
//   B[k][j]: j = l % 16, k = 4 (l / 16) + e
//   D[i][j]: j = l % 16, i = 4 (l / 16) + e
// (checked on the device by amr_cnn_mfma_selftest).  The gfx950 form
// v_mfma_f32_16x16x32_bf16 has twice the K at the same cost: k = 8 (l / 16) + e,
// e = 0..7, D as above.
#pragma once

#include <hip/hip_runtime.h>

namespace amr {
namespace cnnd {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f2bf(float f) {
  // round to nearest even
  unsigned int u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40);  // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

// f2bf by the gfx950 conversion instruction (the same rounding to nearest
// even; a NaN stays a NaN)
__device__ __forceinline__ unsigned short f2bf_hw(float f) {
  const __bf16 h = (__bf16)f;
  return __builtin_bit_cast(unsigned short, h);
}

__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float(((unsigned)h) << 16); }

__device__ __forceinline__ f4 mfma(s4 a, s4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

typedef unsigned u4 __attribute__((ext_vector_type(4)));  // 8 BF16 values
typedef __bf16 b8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f4 mfma32(u4 a, u4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, a),
                                                 __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

// one operand of mfma32 from two of mfma (the K order is free as long as both
// operands have the same)
__device__ __forceinline__ u4 join(s4 a, s4 b) {
  const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
  return u4{x.x, x.y, y.x, y.y};
}

__device__ __forceinline__ s4 load4(const unsigned short* p) {
  // p is 8-byte aligned (4 consecutive channels of one pixel)
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  s4 r;
  r.x = (short)(v.x & 0xffff);
  r.y = (short)(v.x >> 16);
  r.z = (short)(v.y & 0xffff);
  r.w = (short)(v.y >> 16);
  return r;
}

// Transposed LDS read (ds_read_b64_tr_b16): the 16 lanes of a group point at
// the 8-byte pieces of 4 rows of 16 values, lane t at piece t % 4 of row
// t / 4, and lane t receives column t of the 4 rows.  With rows = K and
// columns = the operand's other index that is an MFMA operand from K-major
// storage in one read (the lane order is checked by the weight-gradient
// tests).  p: LDS memory, 8-byte aligned.
__device__ __forceinline__ s4 load4_tr(const unsigned short* p) {
  typedef __attribute__((address_space(3))) s4 lds_s4;
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p);
}

// The next number of a counter in LDS, the same for the whole wave.
__device__ __forceinline__ int take(int* counter) {
  int v = 0;
  if ((threadIdx.x & 63) == 0) v = atomicAdd(counter, 1);
  return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ s4 zero4() {
  s4 r = {0, 0, 0, 0};
  return r;
}

__device__ __forceinline__ s4 pack4(short a, short b, short c, short d) {
  s4 r;
  r.x = a;
  r.y = b;
  r.z = c;
  r.w = d;
  return r;
}

}  // namespace cnnd
}  // namespace amr
