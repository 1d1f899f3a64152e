// Matrix-core operands and products shared by the batch kernels (gfx950).  Not part of the
// public ABI.
#pragma once

#include "ffn_device.h"

namespace ffn {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4_t mfma16(bf16x8_t a, bf16x8_t b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8_t bf8(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

// fp32 weights: the same kernels on v_mfma_f32_16x16x4_f32.  A tile chunk is then 4 fp32 (16
// bytes, as 8 bf16 are), the tokens, z and zval stay fp32, and a k step of four chunks is four
// products: component j of every lane's chunk in product j.  A product adds its terms one after
// the other, so a long range in one accumulator rounds like a serial sum (a call's error against
// 64 bits at d = 3840, d_ff = 14231, r = 480, 16 tokens: 7.9e-7, the vector-ALU kernels' 3.5e-7).
// Every k step of the gate and W_up products is summed from zero, then into its load group's
// sum, then into the running sum; the down product sums every group of 32 rows from zero (3.1e-7).
template <class W>
constexpr bool is_f32() {
  return W::EPC == 4;
}
template <class W>
constexpr int tile_elems() {  // elements of a 16-byte tile chunk
  return is_f32<W>() ? 4 : 8;
}
template <class W>
constexpr uint32_t tok_bytes() {  // bytes of a token's fp32 chunk
  return is_f32<W>() ? 16u : 32u;
}
__device__ __forceinline__ f32x4_t mfma16f(float a, float b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <int I>
struct Int {
  static constexpr int value = I;
};

template <int J>
__device__ __forceinline__ float comp(const uint4& v) {
  return __uint_as_float(J == 0 ? v.x : J == 1 ? v.y : J == 2 ? v.z : v.w);
}

// v = hi + lo with both in bf16 (round to nearest even twice)
__device__ __forceinline__ void split8(const float (&v)[8], bf16x8_t& hi, bf16x8_t& lo) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const __bf16 h = (__bf16)v[j];
    hi[j] = h;
    lo[j] = (__bf16)(v[j] - (float)h);
  }
}

// Chunk j (elements 8j .. 8j + 7) of a loaded 16-byte chunk of W, as 8 bf16: the chunk
// itself for bf16, the codes converted for int8 / int4 (exact: small integers), so that
// quantized rows enter the same bf16 operand tiles.  The row scales are applied to the
// products.
template <class W, int J>
__device__ __forceinline__ uint4 bf16_chunk(const uint4& v) {
  if constexpr (W::EPC == 8) {
    return v;
  } else {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      float a, b;  // elements 8J + 2p and 8J + 2p + 1
      if constexpr (W::EPC == 16) {
        const uint32_t w = d[2 * J + (p >> 1)];
        const int e = 2 * (p & 1);
        a = (float)((int32_t)(w << (24 - 8 * e)) >> 24);
        b = (float)((int32_t)(w << (16 - 8 * e)) >> 24);
      } else {
        const uint32_t w = d[J];
        a = (float)((int32_t)(w << (28 - 8 * p)) >> 28);
        b = (float)((int32_t)(w << (24 - 8 * p)) >> 28);
      }
      // the high halves of both (selector bytes 2, 3 of the second operand, then of the first)
      o[p] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
  }
}
// all W::EPC / 8 of them into consecutive 16-byte slots of an LDS row
template <class W>
__device__ __forceinline__ void put_bf16_chunks(uint4* dst, const uint4& v) {
  dst[0] = bf16_chunk<W, 0>(v);
  if constexpr (W::EPC >= 16) dst[1] = bf16_chunk<W, 1>(v);
  if constexpr (W::EPC >= 32) {
    dst[2] = bf16_chunk<W, 2>(v);
    dst[3] = bf16_chunk<W, 3>(v);
  }
}

// Exchanges 16-bit elements between the lanes of a 16-lane group (ds_read_b64_tr_b16): lane
// 4b + c receives element c of the 8-byte chunks addressed by lanes b, 4 + b, 8 + b and 12 + b.
__device__ __forceinline__ uint2 lds_read_tr16(const char* p) {
  const short4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4_t*)(p));
  return __builtin_bit_cast(uint2, v);
}

}  // namespace
}  // namespace ffn
