// Device helpers shared by the patch-forming kernels (kamera_tridiag.hip,
// kamera_patch.hip): vector types, bf16 rounding and splitting, DPP sums.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kamera_launch.h"

namespace kamera {

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef float f32x16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));

// W's first entry of a unit whose tridiagonal solve failed its checks, until
// the Jacobi kernel that follows on the stream replaces it: a NaN, which no
// solved unit stores (its vectors are checked finite).
constexpr uint16_t kFormFailMark = 0x7FC1;

// two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t form_pack2(float a, float b) {
  const f32x2v v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2v));
}

__device__ __forceinline__ uint16_t to_bf16_rne(float x) { return (uint16_t)(form_pack2(x, 0.0f) & 0xffffu); }

// eight bf16 (element 2q in the low half of word q) from fp32 values
__device__ __forceinline__ u32x4v pack_bf16x8(const float (&x)[8]) {
  u32x4v r;
#pragma unroll
  for (int q = 0; q < 4; ++q) r[q] = form_pack2(x[2 * q], x[2 * q + 1]);
  return r;
}

// x = hi + mid + lo exactly, each part bf16 (RNE): bf16 keeps 8 significant
// bits, so x - hi and x - hi - mid are exact in fp32 and the last remainder
// has at most 8 significant bits left (outside the subnormal range)
__device__ __forceinline__ void split3_bf16x8(const float (&x)[8], u32x4v& hi, u32x4v& mid, u32x4v& lo) {
  float r[8], q[8];
  hi = pack_bf16x8(x);
#pragma unroll
  for (int e = 0; e < 8; ++e)
    r[e] = x[e] - __uint_as_float((e & 1) ? (hi[e >> 1] & 0xffff0000u) : (hi[e >> 1] << 16));
  mid = pack_bf16x8(r);
#pragma unroll
  for (int e = 0; e < 8; ++e)
    q[e] = r[e] - __uint_as_float((e & 1) ? (mid[e >> 1] & 0xffff0000u) : (mid[e >> 1] << 16));
  lo = pack_bf16x8(q);
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// sum over each aligned group of 8 lanes: quad_perm [1,0,3,2], [2,3,0,1],
// then row_half_mirror (lane i <-> 7 - i: the other quad)
__device__ __forceinline__ float sum8(float v) {
  v += dpp_f<0xB1>(v);
  v += dpp_f<0x4E>(v);
  return v + dpp_f<0x141>(v);
}

// 16-byte LDS load of four consecutive floats.
__device__ __forceinline__ f32x4v ld4(const float* p) { return *reinterpret_cast<const f32x4v*>(p); }

__device__ __forceinline__ float lane_f(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

}  // namespace kamera
