// fp32 as the exact sum of three bf16 numbers: x = h + m + l, each the rounding (to nearest) of what the ones before leave, so
// 8 + 8 + 8 bits of the 24.  Exact down to |x| = 2^-110 (below, l reaches the denormals of bf16).
#pragma once
#include "common.h"

namespace prism {
namespace {

typedef float s3_f32x8 __attribute__((ext_vector_type(8)));
typedef __bf16 s3_bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int s3_u32x4 __attribute__((ext_vector_type(4)));

__device__ inline void split3(const float (&x)[8], s3_u32x4 (&p)[3]) {
  s3_f32x8 v, r;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    v[e] = x[e];
    // what would round to infinity keeps the largest finite number as its leading part
    const float big = __uint_as_float(0x7F7F0000u), a = __builtin_fabsf(x[e]);
    r[e] = a > big && a <= __uint_as_float(0x7F7FFFFFu) ? __builtin_copysignf(big, x[e]) : x[e];
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const s3_bf16x8 h = __builtin_convertvector(r, s3_bf16x8);
    p[q] = __builtin_bit_cast(s3_u32x4, h);
    if (q < 2) {
      v -= __builtin_convertvector(h, s3_f32x8);
      r = v;
    }
  }
}

}  // namespace
}  // namespace prism
