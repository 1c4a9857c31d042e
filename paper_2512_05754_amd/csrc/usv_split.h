// fp32 values as sums of three bf16 parts, for products to fp32 accuracy on the bf16 matrix cores: see usv_attn_f32.hip.
#pragma once

#include "usv_attn_bf16.h"

namespace usv {
namespace {

struct Split {  // eight values: x = p[0] + p[1] + p[2], exactly from 2^-110 on
  bf16x8 p[3];
};
__device__ __forceinline__ Split split8(const float (&x)[8]) {
  // pairs throughout: one conversion rounds and packs two values, a shift and a mask take them apart again
  Split s;
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
  for (int part = 0; part < 3; ++part) {
    unsigned w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
      const f32x2 pair = {r[2 * e], r[2 * e + 1]};
      w[e] = __builtin_bit_cast(unsigned, __builtin_convertvector(pair, bf16x2));  // to nearest even
      if (part < 2) {  // (exact)
        r[2 * e] -= __uint_as_float(w[e] << 16);
        r[2 * e + 1] -= __uint_as_float(w[e] & 0xffff0000u);
      }
    }
    typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned u32x4;
    s.p[part] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
  }
  return s;
}

// acc = the largest of |x[0..7]| and acc, NaN left out.  (assembly: without the moves that quiet a NaN ahead of every fmaxf)
__device__ __forceinline__ void largest8(float& acc, const float (&x)[8]) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(acc) : "v"(x[e]), "v"(x[e + 1]));
}

__device__ __forceinline__ f32x4 mfma(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace
}  // namespace usv
