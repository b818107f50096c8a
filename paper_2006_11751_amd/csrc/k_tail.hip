// FC layer, recurrent cell and heads on few rows as one launch (paper, App. "Model architectures").
//
// On few rows each of the three is a launch of 4 to 7 us of which 4 are the launch itself and one trip to
// memory, and each fetches its weights only after the one before has ended.  Here they are roles of the
// workgroups of one launch, on the tiles that k_dense_split.hip and k_heads.hip take for few rows (16 rows
// x 16 outputs, 16 rows x 8 hidden units, 16 rows), with the arithmetic and the order of every sum of
// theirs: the bits are the same.  The features and the new states go from role to role through an
// exchange buffer (sf_exchange.h), which the step's first launch prepares.  What a role needs of its own
// (weights, flags, the incoming state) it asks for before it waits.
//
// Progress.  Roles are numbered level by level: FC tiles, cell tiles, then heads and the state table's writers.  A role
// waits only for roles of lower levels, FC tiles for nobody.  Each workgroup has a role of its own, by its number, and
// marks it as claimed when it starts.  A wait that has lasted a while is given up; the workgroup then looks for a role
// of a lower level that nobody has claimed (the device or the stream's compute units are full of others, so
// that its workgroup has not started), claims it, computes it and begins its own again.  With all of them
// claimed, each is computed by a workgroup that runs, and it waits as long as it takes.  So a wait never
// depends on a workgroup that has not started, however few of them run at a time.  A workgroup that starts
// late and finds its cell tile claimed leaves: the state table may be new by then, since it is written as soon as
// all cell tiles, each computed once, are marked as complete.  An FC tile is computed once more, with the same
// bits, since waiting for the answer to a claim, 2 us with many at a time, would be part of every step.
//
// What many waiting workgroups read over and over holds up the stores that they wait for (a look of all waves at all
// their features, and at the claims first: the features came 3 us later).  So a wave looks at one word of each
// tile that it waits for, with pauses, and then reads them all.
//
// What bounds it at 16 rows in fp32 (13 us): FC tiles 5 (368 KB of operands into each of 32 compute units), two
// exchanges of 1.5 to 2, products, sums and gates of the cell 2, heads and sampler 2.3.
#include <limits.h>

#include <type_traits>

#include "sf_cell.h"
#include "sf_exchange.h"
#include "sf_heads.h"
#include "sf_internal.h"
#include "sf_split.h"

namespace sf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kD = 4;               // K steps in flight of a cell tile
constexpr int kFD = 9;              // ... of an FC tile: all that a wave has of 2304 inputs
constexpr int kP32 = 36, kP16 = 20;  // pitch of a row in LDS (floats)
constexpr int kPatience = 64;        // looks, about 1 us each, before a wait is given up
constexpr unsigned kComplete = 2;    // with a state table: in a cell tile's claim when it is through with the old states

struct TailArgs {
  DenseArgs fc;    // x1, w, b1, M, I1, N, kn; out: exchange buffer of the features
  DenseArgs cell;  // x1: exchange buffer of the features; out: state rows, or null (a state table)
  HeadsArgs heads; // h: exchange buffer of the new states
  unsigned* claims;
  int n_fc, n_cell, n_heads;  // roles; with a state table as many writers of it as heads (8 bytes more here: 0.2 us)
  int fc_cg, cell_cg;         // workgroups along the columns
  int skip;                   // workgroups that leave at once (0; the tests' stand-in for ones that never start)
};

template <int NT>
union TailLds {
  struct {
    float pool[kWaves * 16 * kP32 > kWaves * 3 * 256 ? kWaves * 16 * kP32 : kWaves * 3 * 256];
    int odd_row[16];
    int lost;
  } dense;
  HeadsLds<NT> heads;
  struct {
    int later[16];  // a later row of the batch names the same environment
    int lost;
  } table;
};

template <bool F16>
__device__ inline void mfma(const u32x4& w, const u32x4& x, f32x4& c) {
  if (F16)
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0, 0);
  else
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
}
// The products of one K step and row tile with T tiles of weights in PB terms, smallest first.  ALL: the row
// has three terms.
template <bool ALL, int PB, int T, bool F16>
__device__ inline void products(const u32x4 (&w)[PB][T], const u32x4 (&x)[3], f32x4* acc) {
  auto term = [&](int wq, int xq) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < T; ++t) mfma<F16>(w[wq][t], x[xq], acc[t]);
  };
  if constexpr (ALL && PB == 3) {
    term(2, 0);
    term(0, 2);
    term(1, 1);
    term(1, 0);
    term(0, 1);
  } else if constexpr (ALL) {
    term(0, 2);
    term(0, 1);
  }
  term(0, 0);
}
// A K step's fp32 rows (two 16-byte pieces per lane, eight lanes to a row) through the wave's corner of LDS
// into operand order, in three terms or rounded to one.
template <bool ALL>
__device__ inline void operand(float* turn, int lane, const f32x4 (&a)[2], u32x4 (&x)[3], float& left) {
#pragma unroll
  for (int j = 0; j < 2; ++j) *(f32x4*)(turn + (8 * j + (lane >> 3)) * kP32 + (lane & 7) * 4) = a[j];
  const int at = (lane & 15) * kP32 + (lane >> 4) * 8;
  const f32x4 v0 = *(const f32x4*)(turn + at), v1 = *(const f32x4*)(turn + at + 4);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float e0 = p < 2 ? v0[2 * p] : v1[2 * p - 4], e1 = p < 2 ? v0[2 * p + 1] : v1[2 * p - 3];
    if constexpr (!ALL) {
      const f32x2 e = {e0, e1};
      x[0][p] = __builtin_bit_cast(unsigned, __builtin_convertvector(e, bf16x2));
    } else {
      unsigned t0, t1, t2;
      split_pair(e0, e1, t0, t1, t2, left);
      x[0][p] = t0;
      x[1][p] = t1;
      x[2][p] = t2;
    }
  }
}
// The same of 16-bit rows (one piece per lane, four lanes to a row).
__device__ inline void operand16(float* turn, int lane, const f32x4& a, u32x4 (&x)[3]) {
  *(f32x4*)(turn + (lane >> 2) * kP16 + (lane & 3) * 4) = a;
  x[0] = __builtin_bit_cast(u32x4, *(const f32x4*)(turn + (lane & 15) * kP16 + (lane >> 4) * 4));
}

// One tile of the FC layer: rows 16 rt .., outputs 16 cg ...  claim: the role's mark.
template <int FT, int PB, bool OUT16, typename Lds>
__device__ inline __attribute__((always_inline)) void fc_tile(const DenseArgs& g, int rt, int cg, unsigned* claim, Lds& lds) {
  constexpr bool F32 = FT == X_F32;
  constexpr int NL = F32 ? 2 : 1;
  f32x4(*red)[64] = (f32x4(*)[64])lds.pool;
  const int tid = role_thread(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15;
  const int row0 = 16 * rt;
  if (tid < 16) lds.odd_row[tid] = 0;
  uint32_t row[NL];  // (of few rows: 32-bit offsets from a base in scalar registers)
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int m = min(row0 + (F32 ? 8 * j + (lane >> 3) : lane >> 2), g.M - 1);
    row[j] = (uint32_t)(m * g.I1) * (F32 ? 4 : 2) + (lane & (F32 ? 7 : 3)) * 16;
  }
  const uint8_t* wbase = g.w + (size_t)cg * g.kn * (PB * 1024);
  const uint32_t wat = lane * 16;
  const int s_begin = g.kn * wave / kWaves, s_end = g.kn * (wave + 1) / kWaves;
  f32x4 a[kFD][NL];
  u32x4 b[kFD][PB][1];
  auto load = [&](int i, int s) __attribute__((always_inline)) {
    s = max(min(s, s_end - 1), 0);
#pragma unroll
    for (int j = 0; j < NL; ++j) a[i][j] = *(const f32x4*)((const uint8_t*)g.x1 + (size_t)s * (F32 ? 128 : 64) + row[j]);
#pragma unroll
    for (int p = 0; p < PB; ++p) b[i][p][0] = *(const u32x4*)(wbase + ((size_t)s * PB + p) * 1024 + wat);
  };
  f32x4 acc[1] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
  float left = 0.0f;
  float* turn = lds.pool + wave * (16 * kP32);
  auto use = [&](int i) __attribute__((always_inline)) {
    u32x4 x[3];
    if constexpr (F32)
      operand<true>(turn, lane, a[i], x, left);
    else
      operand16(turn, lane, a[i][0], x);
    products<F32, PB, 1, FT == X_F16>(b[i], x, acc);
  };
#pragma unroll
  for (int i = 0; i < kFD; ++i) load(i, s_begin + i);
  const f32x4 bias = *(const f32x4*)(g.b1 + cg * 16 + (tid & 3) * 4);
  if (tid == 0) store_word(claim, 1u);  // (behind the loads: it is not waited for with them)
  int s = s_begin;
  for (; s + kFD < s_end; s += kFD)
#pragma unroll
    for (int i = 0; i < kFD; ++i) {
      use(i);
      load(i, s + i + kFD);
    }
#pragma unroll
  for (int i = 0; i < kFD; ++i)
    if (s + i < s_end) use(i);
  __syncthreads();  // (the corners are no longer read)
  if (left != left) lds.odd_row[li] = 1;
  red[wave][lane] = acc[0];
  __syncthreads();
  if (tid < 64) {  // thread -> row, four outputs; neighbouring lanes have a row's sixteen
    const int r = tid >> 2, q = tid & 3, m = row0 + r;
    f32x4 v = red[0][q * 16 + r];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += red[w][q * 16 + r];
    bool odd = lds.odd_row[r] != 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) odd |= !finite(v[e]);
    if (__builtin_expect(odd, 0) && m < g.M)
      for (int e = 0; e < 4; ++e) v[e] = plain_sum<FC, FT, PB>(g, m, m, false, 0, cg * 16 + q * 4 + e, 0, g.kn);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e] + bias[e], 0.0f);
    const int at = m * g.N + cg * 16 + q * 4;
    const auto out = __builtin_amdgcn_make_buffer_rsrc(g.out, 0, g.M * g.N * (OUT16 ? 2 : 4), 0x00027000);
    if (m < g.M) {
      if constexpr (OUT16) {
        const f32x2 lo = {v[0], v[1]}, hi = {v[2], v[3]};
        u32x2 pk;
        pk[0] = __builtin_bit_cast(unsigned, __builtin_convertvector(lo, bf16x2));
        pk[1] = __builtin_bit_cast(unsigned, __builtin_convertvector(hi, bf16x2));
        __builtin_amdgcn_raw_buffer_store_b64(pk, out, 2 * at, 0, kDeviceScope);
      } else {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out, 4 * at, 0, kDeviceScope);
      }
    }
  }
}

// One tile of the cell: rows 16 rt .., hidden units 8 cg ...
// False if the wait for the features was given up after `limit` looks (nothing is stored then).
template <int KIND, int XT, int PB, typename Lds>
__device__ inline __attribute__((always_inline)) bool cell_tile(const DenseArgs& g, int rt, int cg, float* states, int limit, Lds& lds) {
  constexpr int GB = group_bytes(KIND), NB = 2, NA = KIND == GRU ? 3 : 2;
  constexpr bool R16 = XT == X_BF16, ALLX = XT == X_F32;
  f32x4(*red)[NA][64] = (f32x4(*)[NA][64])lds.pool;
  const int tid = role_thread(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int row0 = 16 * rt;
  if (tid < 16) lds.odd_row[tid] = 0;
  // rows of the state table: ids[m] where ids are given; an id outside it reads as a zero state
  auto state_row = [&](int m, bool& reset) __attribute__((always_inline)) {
    reset = g.done[m] != 0;
    if (!g.ids) return m;
    const int e = g.ids[m];
    const bool bad = (unsigned)e >= (unsigned)g.n_env;
    reset |= bad;
    return bad ? 0 : e;
  };
  int hm[2];
  bool zero[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) hm[j] = state_row(min(row0 + 8 * j + (lane >> 3), g.M - 1), zero[j]);
  uint32_t woff[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t)  // (GRU: the eight n columns twice)
    woff[t] = KIND == LSTM || t == 0 ? t * 1024 + lane * 16 : 1024 + (lg * 8 + (li & 7)) * 16;
  const uint8_t* wbase = g.w + (size_t)cg * g.kn * (PB * GB);
  const int s_begin = g.kn * wave / kWaves, s_end = g.kn * (wave + 1) / kWaves;
  u32x4 b[kD][PB][NB];
  f32x4 a[kD][2];
  auto load_w = [&](int s0, int s1) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kD; ++i) {
      const int s = min(s0 + i, s1 - 1);
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int t = 0; t < NB; ++t) b[i][p][t] = *(const u32x4*)(wbase + ((size_t)s * PB + p) * GB + woff[t]);
    }
  };
  // thread -> (row, unit), the eight units of a row in neighbouring lanes
  const int er = tid & 3, eq = (tid >> 2) & 1, erow = (tid >> 3) & 15, unit = cg * 8 + eq * 4 + er;
  float bias[2][4] = {}, prev;
  bool greset;
  {
#pragma unroll
    for (int q = 0; q < (KIND == LSTM ? 4 : 3); ++q) {
      bias[0][q] = g.b1[q * g.H + unit];
      bias[1][q] = g.b2[q * g.H + unit];
    }
    const int ghm = state_row(min(row0 + erow, g.M - 1), greset);
    prev = g.h_in[(size_t)ghm * g.S + (KIND == LSTM ? g.H : 0) + unit];
  }
  const auto feat = __builtin_amdgcn_make_buffer_rsrc((void*)g.x1, 0, g.M * g.I1 * (R16 ? 2 : 4), 0x00027000);
  uint32_t xoff[R16 ? 1 : 2];
#pragma unroll
  for (int j = 0; j < (R16 ? 1 : 2); ++j)
    xoff[j] = R16 ? 2u * (uint32_t)(min(row0 + (lane >> 2), g.M - 1) * g.I1 + (lane & 3) * 8)
                  : 4u * (uint32_t)(min(row0 + 8 * j + (lane >> 3), g.M - 1) * g.I1 + (lane & 7) * 4);

  f32x4 acc[NA];
#pragma unroll
  for (int t = 0; t < NA; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  float left = 0.0f;
  float* turn = lds.pool + wave * (16 * kP32);
  // The GRU's n gate needs its sums over the features and over the state apart.
  auto move_n = [&]() __attribute__((always_inline)) {
    if constexpr (KIND == GRU) {
      acc[2] = acc[1];
      acc[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
  };
  // features: until all of a few steps are there
  bool lost = false;
  const int s_mid = max(s_begin, min(s_end, g.k2));
  for (int s0 = s_begin; s0 < s_mid; s0 += kD) {
    load_w(s0, s_mid);
    // a word of each FC tile of these steps (16 features each), in the tile's last row
    const int ahead = 32 * s0 + 16 * min(lane & 7, 2 * (s_mid - s0) - 1);
    const unsigned* word = (const unsigned*)g.x1 + ((size_t)min(row0 + 15, g.M - 1) * g.I1 + ahead) / (R16 ? 2 : 1);
    for (int tries = 0; !lost; ++tries) {
      if (!__any(load_word(word) == kNotYet)) break;
      lost = tries >= limit;
      __builtin_amdgcn_s_sleep(8);
    }
    for (int tries = 0; !lost; ++tries) {
      unsigned missing = 0;
#pragma unroll
      for (int i = 0; i < kD; ++i)
#pragma unroll
        for (int j = 0; j < (R16 ? 1 : 2); ++j) {
          const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(feat, xoff[j], min(s0 + i, s_mid - 1) * (R16 ? 64 : 128), kDeviceScope);
          a[i][j] = __builtin_bit_cast(f32x4, v);
#pragma unroll
          for (int e = 0; e < 4; ++e) missing |= (unsigned)(v[e] == kNotYet);
        }
      if (__all(missing == 0)) break;
      lost = tries >= limit;
      __builtin_amdgcn_s_sleep(4);
    }
#pragma unroll
    for (int i = 0; i < kD; ++i) {
      if (lost || s0 + i >= s_mid) break;
      u32x4 x[3];
      if constexpr (R16)
        operand16(turn, lane, a[i][0], x);
      else
        operand<ALLX>(turn, lane, a[i], x, left);
      products<ALLX, PB, NB, false>(b[i], x, acc);
    }
  }
  if (s_mid == g.k2 || s_end <= g.k2) move_n();
  // the state
  for (int s0 = s_mid; s0 < s_end; s0 += kD) {
    load_w(s0, s_end);
#pragma unroll
    for (int i = 0; i < kD; ++i) {
      const float* from = g.h_in + 32 * (min(s0 + i, s_end - 1) - g.k2) + (lane & 7) * 4;
#pragma unroll
      for (int j = 0; j < 2; ++j) a[i][j] = *(const f32x4*)(from + (size_t)hm[j] * g.S);
    }
#pragma unroll
    for (int i = 0; i < kD; ++i) {
      if (s0 + i >= s_end) break;
      u32x4 x[3];
      const f32x4 none = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int j = 0; j < 2; ++j) a[i][j] = zero[j] ? none : a[i][j];
      operand<true>(turn, lane, a[i], x, left);
      products<true, PB, NB, false>(b[i], x, acc);
    }
  }
  if (lost) lds.lost = 1;
  __syncthreads();
  if (__builtin_expect(lds.lost, 0)) return false;
  if (left != left) lds.odd_row[li] = 1;
#pragma unroll
  for (int t = 0; t < NA; ++t) red[wave][t][lane] = acc[t];
  __syncthreads();
  if (tid < 128) {
    // the gates of one unit: (tile, lane group) of the four sums
    int tl[4], ln[4];
    if (KIND == LSTM) {
      tl[0] = tl[1] = 0;
      tl[2] = tl[3] = 1;
      ln[0] = ln[2] = eq;
      ln[1] = ln[3] = 2 + eq;
    } else {
      tl[0] = tl[1] = 0;
      tl[2] = 2;
      tl[3] = 1;
      ln[0] = eq;
      ln[1] = 2 + eq;
      ln[2] = ln[3] = eq;
    }
    float sum[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float* src = (const float*)&red[0][tl[q]][16 * ln[q] + erow] + er;
      float v = src[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += src[w * (NA * 64 * 4)];
      sum[q] = v;
    }
    const int m = row0 + erow;
    if (m < g.M) {
      bool odd = lds.odd_row[erow] != 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) odd |= !finite(sum[q]);
      if (__builtin_expect(odd, 0)) plain_sums<KIND, XT, PB, true>(g, m, greset, unit, sum);
      const float before = greset ? 0.0f : prev;
      float h, c = 0.0f;
      if (KIND == LSTM)
        h = lstm_gates(sum, bias, before, c);
      else
        h = gru_gates(sum, bias, before);
      unsigned* ex = (unsigned*)states + (size_t)m * g.S + unit;
      store_word(ex, exchange_bits(h));
      if (KIND == LSTM && !g.out) store_word(ex + g.H, exchange_bits(c));
      if (g.out) {
        float* o = (float*)g.out + (size_t)m * g.S + unit;
        o[0] = h;
        if (KIND == LSTM) o[g.H] = c;
      }
    }
  }
  return true;
}

// The new states of rows row0 .. go to the table once all cell tiles have read its old ones, those of other rows, too:
// two rows of the batch may name one environment, and both are computed from its old state.  The last of them leaves
// its state there.  False if the wait was given up after `limit` looks.  Workgroups of their own: done by the heads at
// their end, indexed steps were 1.0 to 1.7 us longer without waiting for other rows' tiles (16 rows of the standard
// network 26.7 us, now 25.0; 60 rows 31.4, 29.9; LSTM, 33 rows 30.8, 29.9), and 0.8 us more with it.
template <typename Lds>
__device__ inline __attribute__((always_inline)) bool table_rows(const HeadsArgs& g, const unsigned* cells, int n_cell, int row0, int limit, Lds& lds) {
  const int tid = role_thread();
  const int rows = min(g.B - row0, 16), r = tid & 15;
  if (tid < 16) lds.later[tid] = 0;
  __syncthreads();
  if (r < rows) {
    const int env = g.ids[row0 + r];
    for (int j = row0 + r + 1 + (tid >> 4); j < g.B; j += kThreads / 16)
      if (g.ids[j] == env) lds.later[r] = 1;
  }
  for (int at = tid; at < n_cell; at += kThreads)
    for (int tries = 0; !(load_word(cells + at) & kComplete); ++tries) {
      if (tries >= limit) {
        lds.lost = 1;
        break;
      }
      __builtin_amdgcn_s_sleep(16);
    }
  __syncthreads();
  if (__builtin_expect(lds.lost, 0)) return false;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)g.h, 0, 4 * g.B * g.S, 0x00027000);
  const int per = g.S / 4;
  constexpr int kPieces = 4;  // in flight (one by one: 2 us more with an LSTM's states)
  for (int i0 = tid; i0 < rows * per; i0 += kPieces * kThreads) {
    u32x4 v[kPieces];
    bool missing;
    do {  // (the tiles are complete: their words are here or on their way)
      missing = false;
#pragma unroll
      for (int u = 0; u < kPieces; ++u) {
        const int i = min(i0 + u * kThreads, rows * per - 1), q = i / per;
        v[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, 4 * ((row0 + q) * g.S + 4 * (i - q * per)), 0, kDeviceScope);
      }
#pragma unroll
      for (int u = 0; u < kPieces; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) missing |= v[u][e] == kNotYet;
    } while (missing);
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      const int i = i0 + u * kThreads, q = i / per;
      if (i >= rows * per) break;
      const uint32_t env = (uint32_t)g.ids[row0 + q];
      if (env < (uint32_t)g.n_env && !lds.later[q]) *((u32x4*)(g.h_table + (size_t)env * g.S) + i - q * per) = v[u];
    }
  }
  return true;
}

// The kernel's argument, each time opaque: a role's part of it is loaded when the role begins.  (Loaded for all
// roles ahead of the loop over them, as the compiler has it otherwise, it does not fit the scalar registers; 190
// of them were spilled to lanes and read back, 2 us of each role.  14 to 20 still are with fp16 rows.)
__device__ inline const TailArgs& tail_args() {
  auto p = (const __attribute__((address_space(4))) TailArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const TailArgs*)p;
}

// TABLE: with a state table (an instantiation of its own: 0.1 to 0.25 us of a step without one).
template <int KIND, int FT, int XT, int PB, int NT, bool TABLE>
__global__ __launch_bounds__(kThreads, 2) void tail_kernel(TailArgs) {
  const TailArgs& g = tail_args();
  __shared__ __attribute__((aligned(16))) TailLds<NT> lds;
  __shared__ int s_run;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int own = (int)blockIdx.x;
  if (own < g.skip) return;
  auto claim = [&](int role) {  // by one lane: whether it is this workgroup's now
    return __hip_atomic_fetch_or(g.claims + role, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
  };
  auto begin = [&](int role) {  // by one thread, ahead of a barrier
    if (role < g.n_fc + g.n_cell)
      lds.dense.lost = 0;
    else if (!TABLE || role < g.n_fc + g.n_cell + g.n_heads)
      lds.heads.lost = 0;
    else
      lds.table.lost = 0;
  };
  if (own >= g.n_fc) {
    if (threadIdx.x == 0) {
      s_run = (TABLE && own >= g.n_fc + g.n_cell + g.n_heads) || claim(own);  // (the table's writers have no claims)
      begin(own);
    }
    __syncthreads();
    if (!s_run) return;
  }
  int run = own, limit = kPatience;
  for (;;) {
    bool complete = true;
    if (run < g.n_fc) {
      const TailArgs& t = tail_args();
      fc_tile<FT, PB, XT == X_BF16>(t.fc, run / t.fc_cg, run % t.fc_cg, t.claims + run, lds.dense);
    } else if (run < g.n_fc + g.n_cell) {
      const TailArgs& t = tail_args();
      const int r = run - t.n_fc;
      complete = cell_tile<KIND, XT, PB>(t.cell, r / t.cell_cg, r % t.cell_cg, (float*)t.heads.h, run == own ? limit : INT_MAX, lds.dense);
      if (TABLE && complete) {
        __syncthreads();  // every wave has stored what it computed from the table
        if (threadIdx.x == 0) store_word(t.claims + run, 1u | kComplete);
      }
    } else if (!TABLE || run < g.n_fc + g.n_cell + g.n_heads) {
      const TailArgs& t = tail_args();
      complete = heads_rows<NT, PB, true>(t.heads, (run - t.n_fc - t.n_cell) * kHeadRows, lds.heads, limit);
    } else {
      const TailArgs& t = tail_args();
      complete = table_rows(t.heads, t.claims + t.n_fc, t.n_cell, (run - t.n_fc - t.n_cell - t.n_heads) * 16, limit, lds.table);
    }
    if (run == own && complete) return;
    __syncthreads();  // LDS is free
    // given up, or back from another role: the first role of a lower level that no one has claimed
    if (wave == 0) {
      const int below = own < g.n_fc + g.n_cell ? g.n_fc : g.n_fc + g.n_cell;
      int role = own;
      for (int at = 0; at < below && role == own; at += 64) {
        unsigned long long open = __ballot(at + lane < below && load_word(g.claims + min(at + lane, below - 1)) == 0);
        while (open && role == own) {
          const int r = at + __builtin_ctzll(open);
          int won = 0;
          if (lane == 0) won = claim(r);
          if (__any(won)) role = r;
          open &= open - 1;
        }
      }
      if (lane == 0) {
        s_run = role;
        begin(role);
      }
    }
    __syncthreads();
    run = __builtin_amdgcn_readfirstlane(s_run);
    if (run == own) limit = INT_MAX;
    __syncthreads();  // (it may be set again)
  }
}

template <int KIND, int FT, int XT, int PB, int NT>
void launch_t(const TailArgs& g, hipStream_t st) {
  const int blocks = g.n_fc + g.n_cell + g.n_heads;
  if (g.heads.h_table)
    tail_kernel<KIND, FT, XT, PB, NT, true><<<blocks + g.n_heads, kThreads, 0, st>>>(g);
  else
    tail_kernel<KIND, FT, XT, PB, NT, false><<<blocks, kThreads, 0, st>>>(g);
}
template <int KIND, int FT, int XT, int PB>
hipError_t launch_nt(const TailArgs& g, hipStream_t st) {
  switch ((g.heads.sumA + 16) / 16) {
    case 1: launch_t<KIND, FT, XT, PB, 1>(g, st); break;
    case 2: launch_t<KIND, FT, XT, PB, 2>(g, st); break;
    case 3: launch_t<KIND, FT, XT, PB, 3>(g, st); break;
    default: launch_t<KIND, FT, XT, PB, 4>(g, st); break;
  }
  return hipGetLastError();
}
template <int FT, int XT, int PB>
hipError_t launch_kind(int lstm, const TailArgs& g, hipStream_t st) {
  return lstm ? launch_nt<LSTM, FT, XT, PB>(g, st) : launch_nt<GRU, FT, XT, PB>(g, st);
}

}  // namespace

// Row tiles of 16 whose cell tiles are one round of workgroups and whose roles fit the claims.  Whole steps, the
// three launches against this one (us):
//   rows                        4            16            32            48            64
//   GRU 512, fp32       28.5, 24.6    29.1, 25.3    29.6, 25.9    30.6, 28.1    31.1, 29.0
//   LSTM 512, fp32      28.6, 25.1    29.5, 25.9    30.3, 26.3    31.3, 29.0    31.6, 29.7
//   GRU 512, bf16       23.1, 20.0    23.6, 20.6    23.8, 20.8    23.9, 21.4    24.5, 21.9
//   GRU 256, fp16 rows  (16, 64, 101, 128 rows) 69.7, 66.6    73.0, 70.0    84.6, 81.6    86.9, 84.8
// Beyond, the tiles of k_dense_split.hip grow with the rows, and a launch more or less matters less.
int tail_max_rows(int fc, int H) {
  int rows = 0;
  for (int rt = 1; rt * (H / 8) <= 256 && rt * (fc / 16 + H / 8 + 1) <= kClaims; ++rt) rows = 16 * rt;
  return rows;
}

// Bytes of the claims and the exchange buffers of a policy.
size_t tail_bytes(int rows, int fc, int S) { return 4 * kClaims + 4 * (size_t)rows * ((size_t)fc + S); }

ExchangePrep tail_prep(void* area, int B, int fc, int S, int out_bf16) {
  ExchangePrep p{};
  p.claims = (unsigned*)area;
  p.fill = (exchange_u32x4*)((uint8_t*)area + 4 * kClaims);
  p.n16 = (int)(((size_t)B * fc * (out_bf16 ? 2 : 4) + (size_t)B * S * 4) / 16);
  return p;
}

// f: the FC layer as for launch_dense_fc, c: the cell as for launch_dense_cell, h: the heads; features of type
// x_type of the cell (0 fp32, 1 bf16, 2 fp32 to be rounded), area: prepared by an earlier launch (tail_prep).
hipError_t launch_tail(const TailCall& t, hipStream_t st) {
  const int rows = t.B, fc = t.fc, S = t.lstm ? 2 * t.H : t.H;
  if (rows <= 0 || rows > tail_max_rows(fc, t.H) || (t.flat % 32) || (fc % 32) || (t.H % 32)) return hipErrorInvalidValue;
  TailArgs g{};
  g.claims = (unsigned*)t.area;
  uint8_t* feat = (uint8_t*)t.area + 4 * kClaims;
  float* states = (float*)(feat + (size_t)rows * fc * (t.x_type == 1 ? 2 : 4));
  g.fc.x1 = t.x; g.fc.w = (const uint8_t*)t.fc_w; g.fc.b1 = t.fc_b; g.fc.out = feat;
  g.fc.M = rows; g.fc.I1 = t.flat; g.fc.N = fc; g.fc.k1 = g.fc.k2 = g.fc.kn = t.flat / 32;
  g.cell.x1 = feat; g.cell.h_in = t.h_in; g.cell.done = t.done; g.cell.ids = t.ids; g.cell.w = (const uint8_t*)t.cell_w;
  g.cell.b1 = t.b_ih; g.cell.b2 = t.b_hh; g.cell.out = t.h_table ? nullptr : t.h_out;
  g.cell.M = rows; g.cell.I1 = fc; g.cell.H = t.H; g.cell.S = S; g.cell.n_env = t.n_env;
  g.cell.k1 = g.cell.k2 = fc / 32; g.cell.kn = g.cell.k2 + t.H / 32;
  HeadsArgs& h = g.heads;
  h.h = states; h.w = (const uint8_t*)t.head_split_w; h.head_w = t.head_w; h.head_b = t.head_b; h.head_off = t.head_off;
  h.actions = t.actions; h.logp = t.logp; h.value = t.value; h.logits = t.logits; h.ids = t.ids; h.h_table = t.h_table;
  h.seed_lo = (uint32_t)t.seed; h.seed_hi = (uint32_t)(t.seed >> 32);
  h.step_lo = (uint32_t)t.step; h.step_hi = (uint32_t)(t.step >> 32);
  h.B = rows; h.H = t.H; h.S = S; h.n_heads = t.n_heads; h.sumA = t.sumA; h.n_env = t.n_env;
  const int n_rt = (rows + 15) / 16;
  g.fc_cg = fc / 16; g.cell_cg = t.H / 8;
  g.n_fc = n_rt * g.fc_cg; g.n_cell = n_rt * g.cell_cg; g.n_heads = n_rt;
  g.skip = t.skip < 0 ? 0 : t.skip < g.n_fc + g.n_cell ? t.skip : g.n_fc + g.n_cell;  // (what the others can take over)
  if (t.fc_type == X_F32) return t.x_type == 0 ? launch_kind<X_F32, X_F32, 3>(t.lstm, g, st) : hipErrorInvalidValue;
  if (t.fc_type == X_BF16)
    return t.x_type == 1 ? launch_kind<X_BF16, X_BF16, 1>(t.lstm, g, st) : hipErrorInvalidValue;
  return t.x_type == 2 ? launch_kind<X_F16, X_ROUND, 1>(t.lstm, g, st) : hipErrorInvalidValue;
}

}  // namespace sf
