// fp32 numbers as sums of three bf16 numbers (device code; see k_dense_split.hip for the arithmetic).
#pragma once

#include <hip/hip_runtime.h>

namespace sf {

typedef float split_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));

// Three terms of two numbers; what is left of them is added to `left`: nothing to speak of, or NaN
// for an infinity, a NaN and what rounds up to an infinity, which have no terms.
__device__ inline void split_pair(float r0, float r1, unsigned& t0, unsigned& t1, unsigned& t2, float& left) {
  const split_f32x2 v0 = {r0, r1};
  t0 = __builtin_bit_cast(unsigned, __builtin_convertvector(v0, split_bf16x2));
  r0 -= __builtin_bit_cast(float, t0 << 16);
  r1 -= __builtin_bit_cast(float, t0 & 0xFFFF0000u);
  const split_f32x2 v1 = {r0, r1};
  t1 = __builtin_bit_cast(unsigned, __builtin_convertvector(v1, split_bf16x2));
  r0 -= __builtin_bit_cast(float, t1 << 16);
  r1 -= __builtin_bit_cast(float, t1 & 0xFFFF0000u);
  const split_f32x2 v2 = {r0, r1};
  t2 = __builtin_bit_cast(unsigned, __builtin_convertvector(v2, split_bf16x2));
  left += r0 + r1;
}

}  // namespace sf
