// Weight codes to bf16 matrix-core operands, shared by the tiled GEMM kernels.
#pragma once
#include "common.hpp"
#include "kernels.hpp"

namespace rlx {
namespace {

// 8 int8 codes (k ascending) -> 8 bf16, exact.
__device__ __forceinline__ bf16x8_t int8x8_to_bf16(uint2 c) {
  const uint32_t w[2] = {c.x, c.y};
  uint32_t o[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float f0 = (float)(int8_t)(w[i] & 0xff), f1 = (float)(int8_t)((w[i] >> 8) & 0xff);
    const float f2 = (float)(int8_t)((w[i] >> 16) & 0xff), f3 = (float)(int8_t)(w[i] >> 24);
    o[2 * i] = __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
    o[2 * i + 1] = __builtin_amdgcn_perm(__float_as_uint(f3), __float_as_uint(f2), 0x07060302u);
  }
  return as_bf16x8(make_uint4(o[0], o[1], o[2], o[3]));
}

// 8 int8 codes (k ascending) -> 8 bf16 of q * s, RNE.
__device__ __forceinline__ bf16x8_t int8x8_scaled_to_bf16(uint2 c, float s) {
  const uint32_t w[2] = {c.x, c.y};
  uint32_t o[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    o[2 * i] = pack_bf16x2((float)(int8_t)(w[i] & 0xff) * s, (float)(int8_t)((w[i] >> 8) & 0xff) * s);
    o[2 * i + 1] = pack_bf16x2((float)(int8_t)((w[i] >> 16) & 0xff) * s, (float)(int8_t)(w[i] >> 24) * s);
  }
  return as_bf16x8(make_uint4(o[0], o[1], o[2], o[3]));
}

// 8 int4 codes (k ascending, low nibble first) -> 8 bf16 of (q - z) * s
// (Int4) or fma(q, s, m) (Int4M, z holding m), RNE: the same arithmetic as
// the whole-group conversions below.
// The low and the high nibbles go to the bytes of two words, each byte to
// fp32 with v_cvt_f32_ubyte; (q - z) * s is formed as fma(q, s, -z s), exact
// in the same way: z s (two f16 significands) needs at most 22 bits, so it is
// exact in fp32 and the fma rounds (q - z) s once, like the product of the
// exact difference.
template <Quant Q>
__device__ __forceinline__ bf16x8_t int4x8_to_bf16(uint32_t c, float s, float z) {
  const uint32_t lo = c & 0x0f0f0f0fu, hi = (c >> 4) & 0x0f0f0f0fu;
  const float zs = Q == Quant::Int4 ? -z * s : z;
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float a = (float)((lo >> (8 * j)) & 0xffu), b = (float)((hi >> (8 * j)) & 0xffu);
    o[j] = pack_bf16x2(fmaf(a, s, zs), fmaf(b, s, zs));
  }
  return as_bf16x8(make_uint4(o[0], o[1], o[2], o[3]));
}

}  // namespace
}  // namespace rlx
