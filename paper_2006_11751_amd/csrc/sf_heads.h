// The heads of 16 rows (device code): k_heads.hip's launch and k_tail.hip.  See k_heads.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "sf_exchange.h"
#include "sf_policy.h"
#include "sf_split.h"

namespace sf {

typedef float heads_f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 heads_bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int heads_u32x4 __attribute__((ext_vector_type(4)));

__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                     uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t m0 = 0xD2511F53u, m1 = 0xCD9E8D57u;
    uint32_t hi0 = __umulhi(m0, c0), lo0 = m0 * c0;
    uint32_t hi1 = __umulhi(m1, c2), lo1 = m1 * c2;
    uint32_t n0 = hi1 ^ c1 ^ k0;
    uint32_t n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

struct HeadsArgs {
  const float* h;         // [B][S], the first H floats of a row
  const uint8_t* w;       // packed weights [NT][H / 32][PB][64][8] (rows past the value head: zeros)
  const float* head_w;    // [sumA + 1][H]
  const float* head_b;    // [sumA + 1]
  const int32_t* head_off;
  int32_t* actions;       // null: logits and value only
  float* logp;
  float* value;
  float* logits;          // or null
  const int32_t* ids;     // or null
  float* h_table;         // or null: row ids[b] receives row b's state
  uint32_t seed_lo, seed_hi, step_lo, step_hi;
  int B, H, S, n_heads, sumA, n_env;
};

constexpr int kHeadWaves = 8;
constexpr int kHeadRows = 16;
constexpr int kHeadThreads = 64 * kHeadWaves;


// The thread's number, opaque: nothing that follows from it is taken out of a loop over roles, where it would
// keep registers through all of them.
__device__ inline int role_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <int NT>
struct HeadsLds {
  static constexpr int P32 = 36;                // pitch of a row (floats)
  static constexpr int TURN = kHeadWaves * kHeadRows * P32, RED = kHeadWaves * NT * 64 * 4;
  static constexpr int LP = NT * 16 + 1;        // pitch of a row of logits
  __attribute__((aligned(16))) float pool[TURN > RED ? TURN : RED];
  float s_lg[kHeadRows][LP], s_pt[kHeadRows][LP], s_lp[kHeadRows][SF_MAX_HEADS];
  int s_off[SF_MAX_HEADS + 1], odd_row[kHeadRows];
  int lost;  // (EX) a wait was given up; zero when heads_rows begins
};

// Rows row0 .. by kHeadThreads threads.  EX: the states are another workgroup's of the same launch (h: the
// exchange buffer); false if the wait for them was given up after `limit` reads (nothing is stored then).
template <int NT, int PB, bool EX>
__device__ inline __attribute__((always_inline)) bool heads_rows(const HeadsArgs& g, int row0, HeadsLds<NT>& lds, int limit = 0) {
  constexpr int P32 = HeadsLds<NT>::P32;
  heads_f32x4(*red)[NT][64] = (heads_f32x4(*)[NT][64])lds.pool;
  const int tid = EX ? role_thread() : (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  if (tid < kHeadRows) lds.odd_row[tid] = 0;
  if (tid <= g.n_heads) lds.s_off[tid] = g.head_off[tid];

  // Gumbel noise: thread -> row, block of four categories of a head (at most 27 blocks)
  const int rows = min(g.B - row0, kHeadRows);
  const int r = tid & 15, b = row0 + r;
  float noise[4] = {};
  int noise_q = tid >> 4, noise_k = 0;
  auto draw = [&]() __attribute__((always_inline)) {
    while (noise_k < g.n_heads && noise_q >= (lds.s_off[noise_k + 1] - lds.s_off[noise_k] + 3) / 4) {
      noise_q -= (lds.s_off[noise_k + 1] - lds.s_off[noise_k] + 3) / 4;
      ++noise_k;
    }
    if (noise_k >= g.n_heads || r >= rows) return;
    // with ids, the row stands for environment ids[b]: that is the sampler's counter word
    const uint32_t env = g.ids ? (uint32_t)g.ids[b] : (uint32_t)b;
    uint32_t wd[4];
    philox4x32_10(env, g.step_lo, g.step_hi, ((uint32_t)noise_k << 16) | (uint32_t)noise_q, g.seed_lo, g.seed_hi, wd);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float u = ((float)(wd[e] >> 9) + 0.5f) * 0x1.0p-23f;
      noise[e] = -logf(-logf(u));
    }
  };
  if constexpr (EX) {  // while the states are on their way
    __syncthreads();
    draw();
  }

  const int kn = g.H / 32;
  const int s_begin = kn * wave / kHeadWaves, s_end = kn * (wave + 1) / kHeadWaves;
  // rows with eight lanes side by side on a K step, turned into operand order in the wave's corner
  // of LDS; two K steps in flight
  const uint8_t* src[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    src[j] = (const uint8_t*)(g.h + (size_t)min(row0 + 8 * j + (lane >> 3), g.B - 1) * g.S) + (lane & 7) * 16;
  float* turn = lds.pool + wave * (kHeadRows * P32);
  float head_b[4];  // of the outputs that this thread finishes, where it does
#pragma unroll
  for (int e = 0; e < 4; ++e) head_b[e] = g.head_b[min((tid >> 6) * 16 + 4 * lg + e, g.sumA)];
  heads_f32x4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = heads_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  float left = 0.0f;
  bool lost = false;
  for (int s0 = s_begin; s0 < s_end; s0 += 2) {
    heads_f32x4 a[2][2];
    heads_u32x4 b[2][PB][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int s = min(s0 + u, s_end - 1);
      if constexpr (!EX)
#pragma unroll
        for (int j = 0; j < 2; ++j) a[u][j] = *(const heads_f32x4*)(src[j] + (size_t)s * 128);
#pragma unroll
      for (int q = 0; q < PB; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t) b[u][q][t] = *(const heads_u32x4*)(g.w + (((size_t)t * kn + s) * PB + q) * 1024 + lane * 16);
    }
    if constexpr (EX) {  // until all of them are there
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)g.h, 0, 4 * g.B * g.S, 0x00027000);
      for (int tries = 0; !lost; ++tries) {
        unsigned missing = 0;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const heads_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(src[j] - (const uint8_t*)g.h), 128 * min(s0 + u, s_end - 1), kDeviceScope);
            a[u][j] = __builtin_bit_cast(heads_f32x4, v);
#pragma unroll
            for (int e = 0; e < 4; ++e) missing |= (unsigned)(v[e] == kNotYet);
          }
        if (__all(missing == 0)) break;
        lost = tries >= limit;
        __builtin_amdgcn_s_sleep(8);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (s0 + u >= s_end) break;
#pragma unroll
      for (int j = 0; j < 2; ++j) *(heads_f32x4*)(turn + (8 * j + (lane >> 3)) * P32 + (lane & 7) * 4) = a[u][j];
      const heads_f32x4 v0 = *(const heads_f32x4*)(turn + li * P32 + lg * 8), v1 = *(const heads_f32x4*)(turn + li * P32 + lg * 8 + 4);
      heads_u32x4 x[3];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        unsigned t0, t1, t2;
        split_pair(p < 2 ? v0[2 * p] : v1[2 * p - 4], p < 2 ? v0[2 * p + 1] : v1[2 * p - 3], t0, t1, t2, left);
        x[0][p] = t0;
        x[1][p] = t1;
        x[2][p] = t2;
      }
      auto term = [&](int wq, int xq) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(heads_bf16x8, b[u][wq][t]),
                                                           __builtin_bit_cast(heads_bf16x8, x[xq]), acc[t], 0, 0, 0);
      };
      if constexpr (PB == 3) {
        term(2, 0);
        term(0, 2);
        term(1, 1);
        term(1, 0);
      } else {
        term(0, 2);
      }
      term(0, 1);
      term(0, 0);
    }
  }
  if constexpr (EX) {
    if (lost) lds.lost = 1;
    __syncthreads();
    if (__builtin_expect(lds.lost, 0)) return false;
  } else {
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) red[wave][t][lane] = acc[t];
  if (left != left) lds.odd_row[li] = 1;
  __syncthreads();
  if (tid < NT * 64) {  // sums in wave order: thread -> row li, four outputs
    heads_f32x4 v = red[0][tid >> 6][lane];
#pragma unroll
    for (int w = 1; w < kHeadWaves; ++w) v += red[w][tid >> 6][lane];
    bool odd = lds.odd_row[li] != 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) odd |= !(fabsf(v[e]) < INFINITY);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int a = (tid >> 6) * 16 + 4 * lg + e;
      const int ac = min(a, g.sumA);
      if (__builtin_expect(odd, 0)) {  // an infinity or a NaN in the state or as a sum: plain arithmetic
        const float* hr = g.h + (size_t)min(row0 + li, g.B - 1) * g.S;
        float sum = 0.0f;
        for (int k = 0; k < g.H; ++k) sum = fmaf(EX ? load_float(hr + k) : hr[k], g.head_w[(size_t)ac * g.H + k], sum);
        v[e] = sum;
      }
      lds.s_lg[li][a] = v[e] + head_b[e];
    }
  }
  __syncthreads();
  // value and logits, by the threads from `from` on (with a sampler behind: those that it leaves free)
  auto put = [&](int from) __attribute__((always_inline)) {
    const int t = tid - from;
    if (t < 0) return;
    if (t < rows) g.value[row0 + t] = lds.s_lg[t][g.sumA];
    if (g.logits)
      for (int i = t; i < rows * g.sumA; i += kHeadThreads - from) {
        const int r = i / g.sumA;
        g.logits[(size_t)row0 * g.sumA + i] = lds.s_lg[r][i - r * g.sumA];
      }
  };
  if (!g.actions) {  // (the learner's pass wants logits and value only)
    put(0);
    return true;
  }

  if constexpr (!EX) draw();
  if (noise_k < g.n_heads && r < rows) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int idx = lds.s_off[noise_k] + 4 * noise_q + e;
      if (idx < lds.s_off[noise_k + 1]) lds.s_pt[r][idx] = lds.s_lg[r][idx] + noise[e];
    }
  }
  __syncthreads();
  // thread -> row, head: categories in ascending order, so that the first maximum wins ties
  put(16 * SF_MAX_HEADS);
  const int k = tid >> 4;
  if (k < g.n_heads && r < rows) {
    const int off = lds.s_off[k], A = lds.s_off[k + 1] - off;
    const float *pt = &lds.s_pt[r][off], *l = &lds.s_lg[r][off];
    float best = pt[0], lmax = l[0];
    int arg = 0;
#pragma unroll 4
    for (int i = 1; i < A; ++i) {
      const float pert = pt[i];
      if (pert > best) {
        best = pert;
        arg = i;
      }
      lmax = fmaxf(lmax, l[i]);
    }
    float se = 0.0f;
#pragma unroll 4
    for (int i = 0; i < A; ++i) se += expf(l[i] - lmax);
    lds.s_lp[r][k] = l[arg] - (lmax + logf(se));
    g.actions[(size_t)b * g.n_heads + k] = arg;
  }
  __syncthreads();
  if (tid < rows) {
    float lp = 0.0f;
    for (int q = 0; q < g.n_heads; ++q) lp += lds.s_lp[tid][q];
    g.logp[row0 + tid] = lp;
  }
  return true;
}

}  // namespace sf
