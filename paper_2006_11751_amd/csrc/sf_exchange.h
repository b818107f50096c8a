// What workgroups of one launch hand to one another through memory (device code; k_tail.hip, k_core_seq.hip).
//
// A word is its own flag: the buffer is filled ahead, by an earlier launch, with a bit pattern that no
// value has; values are stored and read with device scope, past the caches that are not coherent across
// the XCDs, and a reader repeats its read until the pattern is gone.  No counters, no fences, no cache
// write-back.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sf {

typedef unsigned int exchange_u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kNotYet = 0xFFFFFFFFu;  // a NaN whose bits are all ones
// cache policy of a buffer access: sc1 (device scope), volatile (repeated as often as it is written)
constexpr int kDeviceScope = (int)0x80000010;

__device__ inline unsigned load_word(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float load_float(const float* p) { return __builtin_bit_cast(float, load_word((const unsigned*)p)); }
__device__ inline void store_word(unsigned* p, unsigned v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a value that may be any NaN: another NaN for the one that is the pattern
__device__ inline unsigned exchange_bits(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  return u == kNotYet ? 0x7FC00000u : u;
}

// Work of an earlier launch for a later one: n16 pieces of 16 bytes to be filled with the pattern, and
// kClaims words to be cleared.
constexpr int kClaims = 512;
struct ExchangePrep {
  unsigned* claims;      // null: nothing to do
  exchange_u32x4* fill;
  int n16;
  bool done;             // (host) a launch has taken it over
};
// by thread `at` of `threads` of the launch
__device__ inline void exchange_prepare(const ExchangePrep& p, int at, int threads) {
  if (!p.claims) return;
  for (int i = at; i < kClaims; i += threads) p.claims[i] = 0;
  const exchange_u32x4 v = {kNotYet, kNotYet, kNotYet, kNotYet};
  for (int i = at; i < p.n16; i += threads) p.fill[i] = v;
}

}  // namespace sf
