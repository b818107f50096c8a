// Fully connected layer and recurrent cell (GRU / LSTM) on the 16-bit matrix instructions with the
// precision of fp32 operands (paper, App. "Model architectures": the FC layer and the core).
//
// Arithmetic.  An fp32 number is the sum of three bf16 numbers (8 + 8 + 8 significant bits, each
// the rounded remainder of the one before), so x * w is the sum of nine exact products.  The six
// largest are kept: x0w0, x0w1, x1w0, x1w1, x0w2, x2w0; what is dropped is at most 2^-23 of the
// product and 2^-27 root mean square, less than the rounding of one fp32 addition.  They run on v_mfma_f32_16x16x32_bf16
// with fp32 accumulators, smallest products first: 16 times the rate of the fp32 matrix
// instructions, over six products.  One instruction adds 32 terms to an accumulator, so a sum is
// rounded 6 times per 32 terms instead of 16 times and comes out nearer to the exact one.  In
// bf16 configurations the weights are bf16 numbers (one term), and the state enters with all three
// terms (three products).  The features are activations of 16 bits there: in the step they are
// bf16 numbers (one product), as they come from the FC layer or rounded here (X_ROUND), as
// k_rnn_bf16.hip, which takes larger batches, rounds them; in the pass over trajectories fp32
// features keep all their bits.
//
// Work split.  What bounds these layers is getting the operands into the registers: with few rows
// the latency of a chain of loads, with many the path from the L2.  So there is no barrier in the K
// loop: a workgroup of eight waves owns 16*RT rows and 8*U hidden units (FC: 16*U outputs), each
// wave an eighth of K, its loads running ahead of the products.  The weights are packed in operand
// order, split ahead of time, and go straight into the registers of the lane that feeds them; the
// rows are turned into operand order and split into their terms on the way.  The eight partial sums meet in LDS and are added in wave order, where the bias and the gates follow.
// The order of every sum depends on K alone: the result of a row is the same bits for every choice
// of RT and U, so these follow the number of rows of the call.  (cell_tile_kernel below, for many
// rows, sums in another order; which of the two a policy uses is settled at create.)
//
// v_mfma_f32_16x16x32_*: lane l supplies A[i = l%16][k = 8*(l/16) + e] and B[k][j = l%16], e = 0..7
// (16 bytes each); D[i][j] sits in lane j + 16*(i/4), register i%4.  A = weights (i = output
// column), B = rows: a lane ends up with four neighbouring outputs of one row.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <type_traits>

#include "sf_cell.h"
#include "sf_internal.h"
#include "sf_meas.h"
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

// Rows of the state table: ids[m] where ids are given; an id outside the table reads as a zero
// state, as after a reset (flag).  One branch for all rows, behind their flag loads: a branch per
// row makes every row wait for the one before.
template <int N>
__device__ inline void state_rows(const DenseArgs& g, int (&row)[N], int (&flag)[N]) {
  if (!g.ids) return;
#pragma unroll
  for (int j = 0; j < N; ++j) row[j] = g.ids[row[j]];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const bool bad = (unsigned)row[j] >= (unsigned)g.n_env;
    flag[j] |= bad;
    row[j] = bad ? 0 : row[j];
  }
}

// Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2: an XCD gets a block of
// neighbouring row tiles and column groups (deal(), below).
__device__ inline bool tile_of(const DenseArgs& g, int& rt, int& cg) {
  const uint32_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int i = (int)(g.per_cg == 1 ? slot : __umulhi(slot, g.rcp_cg));  // slot / per_cg
  rt = (int)(xcd & ((1u << g.xcd_rows) - 1)) * g.per_rt + i;
  cg = (int)(xcd >> g.xcd_rows) * g.per_cg + (int)slot - i * g.per_cg;
  return rt < g.n_rt && cg < g.n_cg;
}

// DA, DB: K steps of rows / weights a wave has in flight; DA = 1: in turn with a second workgroup of the CU, or
// for want of registers.
// MEAS: with workgroups of the measurement layers (an instantiation of its own: 0.2 us of 24 at 60 rows).
template <int KIND, int XT, int PB, int RT, int U, int DA, int DB, bool OUT16, bool MEAS>
__global__ __launch_bounds__(kThreads, DA == 1 && RT * U <= 4 ? 4 : 2) void dense_split_kernel(DenseArgs g) {
  constexpr int GB = group_bytes(KIND);
  constexpr int UN = (U + 1) / 2;                                   // GRU: tiles of n columns
  constexpr int NB = KIND == FC ? U : KIND == GRU ? U + UN : 2 * U;  // weight tiles per K step and term
  constexpr int NA = KIND == FC ? U : KIND == GRU ? U + 2 * UN : 2 * U;  // accumulators per row tile
  constexpr bool LATE = DA == 1;
  constexpr int R16 = 0, R32 = 1, R32_ONE = 2;                      // kinds of rows of a K step: see load_a
  constexpr int RR = RT * NA <= 8 ? RT : 8 / NA;                    // row tiles per round of the sum
  static_assert(KIND == FC || RR * U <= 4, "a thread per unit");
  static_assert(RT % RR == 0, "whole rounds");
  constexpr int TURN = kWaves * 16 * RT * 36, RED = kWaves * RR * NA * 64 * 4;  // floats
  __shared__ __attribute__((aligned(16))) float lds[TURN > RED ? TURN : RED];
  __shared__ int odd_row[16 * RT];  // rows with an infinity or a NaN
  f32x4(*red)[RR * NA][64] = (f32x4(*)[RR * NA][64])lds;  // after the K loop

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  if constexpr (MEAS)
    if ((int)blockIdx.x >= g.blocks) {  // the measurement layers (kMeasThreads threads)
      meas_rows(g.meas, (int)blockIdx.x - g.blocks, lds);
      return;
    }
  int rt0, cg;
  if (!tile_of(g, rt0, cg)) return;
  const int row0 = rt0 * 16 * RT;

  // Rows are loaded with neighbouring lanes on neighbouring bytes (fp32: eight lanes per row, 128
  // bytes = a K step; 16 bits: four lanes, 64 bytes) and turned into operand order in LDS, in a
  // corner of the wave's own: no barrier.  Loaded in operand order (lane = row) the same bytes take
  // 2.5 times as long: 9.6 against 24 TB/s out of the L2, contiguous weights 32.
  // Row indices of this lane's loads (past the end: the last row again, never stored).
  constexpr int NL = 2 * RT;                       // loads per K step of fp32 rows
  if (tid < 16 * RT) odd_row[tid] = 0;
  int xm[NL], hm[NL], dn[NL] = {}, xm16[in_f32(XT) ? 1 : RT];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    xm[j] = hm[j] = min(row0 + 8 * j + (lane >> 3), g.M - 1);
    if (KIND != FC) dn[j] = g.done[xm[j]];
  }
  if (KIND != FC) state_rows(g, hm, dn);
  if (!in_f32(XT))
#pragma unroll
    for (int j = 0; j < RT; ++j) xm16[j] = min(row0 + 16 * j + (lane >> 2), g.M - 1);
  // this lane's place in the weights of a K step: tile t, lane offset
  const size_t group_stride = (size_t)g.kn * PB * GB;
  const uint8_t* wbase = g.w + (size_t)cg * U * group_stride;
  uint32_t woff[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    if (KIND == FC)
      woff[t] = (uint32_t)(t * group_stride) + lane * 16;
    else if (KIND == LSTM)
      woff[t] = (uint32_t)((t >> 1) * group_stride) + (t & 1) * 1024 + lane * 16;
    else if (t < U)
      woff[t] = (uint32_t)(t * group_stride) + lane * 16;
    else  // the n columns: 8 per group (one group: twice the same eight)
      woff[t] = (uint32_t)((U == 1 ? 0 : 2 * (t - U) + (li >> 3)) * group_stride) + 1024 + (lg * 8 + (li & 7)) * 16;
  }

  f32x4 acc[RT][NA];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int t = 0; t < NA; ++t) acc[r][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // What the gates need from memory, requested behind the first operands (LATE: behind the last, for
  // want of registers).  Thread -> (element of four
  // neighbouring outputs, row, four outputs); EPT such elements of a round's row tiles
  constexpr int ET = 16 * 8 * U;               // cells: threads per row tile
  const int er = tid & 3, erow = (tid >> 2) & 15, eq = (tid >> 6) & (2 * U - 1), ert = tid / ET;
  const int unit = (cg * U * 2 + eq) * 4 + er;
  float bias[2][4] = {}, prev[RT / RR] = {};
  int gdn[RT / RR] = {};
  f32x4 fbias = {0, 0, 0, 0};
  constexpr int ft_per_rt = 64 * U;            // FC: threads per row tile
  auto load_gates = [&]() __attribute__((always_inline)) {
    if (KIND == FC) {
      fbias = *(const f32x4*)(g.b1 + cg * 16 * U + ((tid >> 6) % U) * 16 + 4 * lg);
    } else {
  #pragma unroll
      for (int q = 0; q < (KIND == LSTM ? 4 : 3); ++q) {
        bias[0][q] = g.b1[q * g.H + unit];
        bias[1][q] = g.b2[q * g.H + unit];
      }
      int ghm[RT / RR];
  #pragma unroll
      for (int rd = 0; rd < RT / RR; ++rd) {
        ghm[rd] = min(row0 + 16 * (rd * RR + (ert < RR ? ert : 0)) + erow, g.M - 1);
        gdn[rd] = g.done[ghm[rd]];
      }
      state_rows(g, ghm, gdn);
  #pragma unroll
      for (int rd = 0; rd < RT / RR; ++rd) prev[rd] = g.h_in[(size_t)ghm[rd] * g.S + (KIND == LSTM ? g.H : 0) + unit];
    }
  };
  const int s_begin = g.kn * wave / kWaves, s_end = g.kn * (wave + 1) / kWaves;
  f32x4 a[DA][NL];
  u32x4 b[DB][PB][NB];
  auto load_b = [&](auto slotc, int s) __attribute__((always_inline)) {
    constexpr int SL = decltype(slotc)::value;
    s = max(min(s, s_end - 1), 0);
    const uint8_t* wp = wbase + (size_t)s * (PB * GB);
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
      for (int t = 0; t < NB; ++t) b[SL][p][t] = *(const u32x4*)(wp + (woff[t] + p * GB));
  };
  // Rows as 16-bit features, or one of the fp32 pieces (the row pitches are whole K steps) with all
  // terms or with one.
  // (selects, not branches: a branch around a load makes the compiler wait for all loads where
  // the paths join)
  auto load_a = [&](auto kindc, auto slotc, int s) __attribute__((always_inline)) {
    constexpr int SL = decltype(slotc)::value;
    s = max(min(s, s_end - 1), 0);
    if constexpr (decltype(kindc)::value != R16) {
      const uint8_t* base = (const uint8_t*)g.x1 + (size_t)s * 128;
      uint32_t pitch = (uint32_t)g.I1 >> 5;
      if (KIND != FC) {
        base = in_f32(XT) && s < g.k1 ? base : (s < g.k2 ? (const uint8_t*)g.x2 + (size_t)(s - g.k1) * 128
                                                          : (const uint8_t*)g.h_in + (size_t)(s - g.k2) * 128);
        pitch = (uint32_t)(in_f32(XT) && s < g.k1 ? g.I1 : s < g.k2 ? g.I2 : g.S) >> 5;
      }
      base += (lane & 7) * 16;
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        const uint32_t m = KIND == FC || s < g.k2 ? xm[j] : hm[j];
        a[SL][j] = *(const f32x4*)(base + ((size_t)(m * pitch) << 7));
      }
    } else {
      const uint8_t* base = (const uint8_t*)g.x1 + (size_t)s * 64 + (lane & 3) * 16;
#pragma unroll
      for (int j = 0; j < RT; ++j) a[SL][j] = *(const f32x4*)(base + ((size_t)((uint32_t)xm16[j] * ((uint32_t)g.I1 >> 5)) << 6));
    }
  };
  auto mfma = [&](const u32x4& w, const u32x4& x, f32x4& c) __attribute__((always_inline)) {
    if (XT == X_F16)
      c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0, 0);
    else
      c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
  };
  // one K step
  constexpr int P32 = 36, P16 = 20;  // pitch of a row in LDS (floats): 16-byte accesses without conflicts
  float left[RT] = {};
  float* turn = lds + wave * (16 * RT * P32);
  auto use = [&](auto kindc, auto slota, auto slotb, bool state) __attribute__((always_inline)) {
    constexpr int SA = decltype(slota)::value, SB = decltype(slotb)::value;
    constexpr bool F32 = decltype(kindc)::value != R16, TERMS = decltype(kindc)::value == R32;
    if constexpr (F32) {
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        f32x4 v = a[SA][j];
        if (KIND != FC) {
          const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
          v = state && dn[j] ? zero : v;
        }
        *(f32x4*)(turn + (8 * j + (lane >> 3)) * P32 + (lane & 7) * 4) = v;
      }
    } else {
#pragma unroll
      for (int j = 0; j < RT; ++j) *(f32x4*)(turn + (16 * j + (lane >> 2)) * P16 + (lane & 3) * 4) = a[SA][j];
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      u32x4 x[3];
      if (F32) {
        const f32x4 v0 = *(const f32x4*)(turn + (16 * r + li) * P32 + lg * 8);
        const f32x4 v1 = *(const f32x4*)(turn + (16 * r + li) * P32 + lg * 8 + 4);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const float e0 = p < 2 ? v0[2 * p] : v1[2 * p - 4], e1 = p < 2 ? v0[2 * p + 1] : v1[2 * p - 3];
          if constexpr (!TERMS) {
            const f32x2 e = {e0, e1};
            x[0][p] = __builtin_bit_cast(unsigned, __builtin_convertvector(e, bf16x2));
            continue;
          }
          unsigned t0, t1, t2;
          split_pair(e0, e1, t0, t1, t2, left[r]);
          x[0][p] = t0;
          x[1][p] = t1;
          x[2][p] = t2;
        }
      } else {
        x[0] = __builtin_bit_cast(u32x4, *(const f32x4*)(turn + (16 * r + li) * P16 + lg * 4));
      }
      // smallest products first
      if constexpr (TERMS && PB == 3) {
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][2][t], x[0], acc[r][t]);
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][0][t], x[2], acc[r][t]);
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][1][t], x[1], acc[r][t]);
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][1][t], x[0], acc[r][t]);
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][0][t], x[1], acc[r][t]);
      } else if constexpr (TERMS) {
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][0][t], x[2], acc[r][t]);
#pragma unroll
        for (int t = 0; t < NB; ++t) mfma(b[SB][0][t], x[1], acc[r][t]);
      }
#pragma unroll
      for (int t = 0; t < NB; ++t) mfma(b[SB][0][t], x[0], acc[r][t]);
    }
  };
  // The GRU's n gate needs its sums over the features and over the state apart: at the border
  // the first moves aside (acc[U ..] -> acc[U + UN ..]) and acc[U ..] starts again.
  auto move_n = [&]() __attribute__((always_inline)) {
    if constexpr (KIND == GRU) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = U; t < U + UN; ++t) {
          acc[r][t + UN] = acc[r][t];
          acc[r][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
  };
  auto each = [&](auto f) __attribute__((always_inline)) {
    f(std::integral_constant<int, 0>{});
    if constexpr (DA > 1) f(std::integral_constant<int, 1>{});
    if constexpr (DA > 2) f(std::integral_constant<int, 2>{});
    if constexpr (DA > 3) f(std::integral_constant<int, 3>{});
  };
  static_assert(DA % DB == 0, "weights of a step sit in slot (step % DB)");
  // K steps [s0, s1) on rows of one kind.  Steps in flight are refilled without conditions around
  // the loads, then come the last DA without loads.
  auto phase = [&](auto kindc, int s0, int s1) __attribute__((always_inline)) {
    if (s0 >= s1) {
      if (XT == X_F32 && !LATE) load_gates();
      return;
    }
    auto step = [&](auto slota, auto slotb, int s) __attribute__((always_inline)) {
      if (s >= s1) return;
      if (KIND == GRU && s == g.k2) move_n();
      use(kindc, slota, slotb, KIND != FC && s >= g.k2);
    };
    int s = s0;
    each([&](auto i) __attribute__((always_inline)) {
      constexpr int I = decltype(i)::value;
      load_a(kindc, i, s + I);
      if constexpr (I < DB) load_b(i, s + I);
    });
    if (XT == X_F32 && !LATE) load_gates();
    for (; s + DA < s1; s += DA)
      each([&](auto i) __attribute__((always_inline)) {
        constexpr int I = decltype(i)::value;
        using SB = std::integral_constant<int, I % DB>;
        step(i, SB{}, s + I);
        load_b(SB{}, s + I + DB);
        load_a(kindc, i, s + I + DA);
      });
    each([&](auto i) __attribute__((always_inline)) {
      constexpr int I = decltype(i)::value;
      using SB = std::integral_constant<int, I % DB>;
      step(i, SB{}, s + I);
      if constexpr (I + DB < DA) load_b(SB{}, s + I + DB);
    });
  };
  if (XT != X_F32 && !LATE) load_gates();
  using All = std::integral_constant<int, R32>;
  using One = std::integral_constant<int, R32_ONE>;
  if (XT == X_F32) {
    phase(All{}, s_begin, s_end);
  } else if (XT == X_ROUND) {
    phase(One{}, s_begin, min(s_end, g.k2));
    phase(All{}, max(s_begin, g.k2), s_end);
  } else {
    phase(std::integral_constant<int, R16>{}, s_begin, min(s_end, g.k1));
    if (KIND != FC) phase(All{}, max(s_begin, g.k1), s_end);
  }
  if (KIND == GRU && s_end <= g.k2) move_n();
  if (LATE) load_gates();
  // The eight partial sums, RR row tiles at a time, added in wave order.
#pragma unroll
  for (int rd = 0; rd < RT / RR; ++rd) {
    __syncthreads();  // (the K loop's LDS, or the last round's sums, are no longer read)
    if (rd == 0)
#pragma unroll
      for (int r = 0; r < RT; ++r)
        if (left[r] != left[r]) odd_row[16 * r + li] = 1;
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
      for (int t = 0; t < NA; ++t) red[wave][r * NA + t][lane] = acc[rd * RR + r][t];
    __syncthreads();
    if (KIND == FC) {
      for (int u = tid; u < RR * ft_per_rt; u += kThreads) {
        const int r = u / ft_per_rt, t = (u >> 6) % U;
        f32x4 v = red[0][r * NA + t][lane];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += red[w][r * NA + t][lane];
        const int m = row0 + 16 * (rd * RR + r) + li;
        bool odd = odd_row[16 * (rd * RR + r) + li] != 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) odd |= !finite(v[e]);
        if (__builtin_expect(odd, 0) && m < g.M)
          for (int e = 0; e < 4; ++e)
            v[e] = plain_sum<KIND, XT, PB>(g, m, m, false, 0, cg * 16 * U + t * 16 + 4 * lg + e, 0, g.kn);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e] + fbias[e], 0.0f);
        const size_t o = (size_t)m * g.N + cg * 16 * U + t * 16 + 4 * lg;
        if (m < g.M) {
          if (OUT16) {
            const f32x2 lo = {v[0], v[1]}, hi = {v[2], v[3]};
            u32x2 pk;
            pk[0] = __builtin_bit_cast(unsigned, __builtin_convertvector(lo, bf16x2));
            pk[1] = __builtin_bit_cast(unsigned, __builtin_convertvector(hi, bf16x2));
            *(u32x2*)((uint16_t*)g.out + o) = pk;
          } else {
            *(f32x4*)((float*)g.out + o) = v;
          }
        }
      }
    } else {
      if (ert < RR) {
        // the gates of one unit: (tile, lane group) of the four sums
        const int gq = eq >> 1, hq = eq & 1;
        int tl[4], ln[4];
        if (KIND == LSTM) {
          tl[0] = tl[1] = 2 * gq;
          tl[2] = tl[3] = 2 * gq + 1;
          ln[0] = ln[2] = hq;
          ln[1] = ln[3] = 2 + hq;
        } else {
          tl[0] = tl[1] = gq;
          tl[2] = U + UN + (eq >> 2);
          tl[3] = U + (eq >> 2);
          ln[0] = hq;
          ln[1] = 2 + hq;
          ln[2] = ln[3] = eq & 3;
        }
        float sum[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float* src = (const float*)&red[0][ert * NA + tl[q]][16 * ln[q] + erow] + er;
          float v = src[0];
#pragma unroll
          for (int w = 1; w < kWaves; ++w) v += src[w * (RR * NA * 64 * 4)];
          sum[q] = v;
        }
        const int m = row0 + 16 * (rd * RR + ert) + erow;
        if (m < g.M) {
          float* o = (float*)g.out + (size_t)m * g.S;
          const bool rs = gdn[rd] != 0;
          bool odd = odd_row[16 * (rd * RR + ert) + erow] != 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) odd |= !finite(sum[q]);
          if (__builtin_expect(odd, 0))
            plain_sums<KIND, XT, PB>(g, m, rs, unit, sum);
          const float before = rs ? 0.0f : prev[rd];
          if (KIND == LSTM)
            cell_lstm(o, g.H, unit, sum, bias, before);
          else
            cell_gru(o, unit, sum, bias, before);
        }
      }
    }
  }
}

// The cell of an fp32 configuration in handles for many rows: a workgroup owns 16 * RT rows (64; fewer in calls of
// few, see launch_tile: the bits of a row are the same) and 32 hidden units in two halves.  Four waves share a half and take every fourth K step; the rows of a chunk of four K
// steps are split once for all eight waves and wait in LDS in operand order (two buffers, one
// barrier per chunk), the weights go from memory to the one wave that needs them.
template <int KIND, int RT>
__global__ __launch_bounds__(kThreads, 2) void cell_tile_kernel(DenseArgs g) {
  constexpr int XT = X_F32, PB = 3;
  constexpr int GB = group_bytes(KIND);
  constexpr int U = 2;                         // column groups per wave
  constexpr int NB = KIND == GRU ? U + 1 : 2 * U, NA = 2 * U;
  constexpr int KW = 4;                        // K steps per chunk
  constexpr int RR = RT < 2 ? 1 : 2;           // row tiles per round of the sum
  constexpr int NP = 3;                        // terms of a row element
  constexpr int BUF = NP * RT * KW * 1024;     // bytes of a chunk in LDS
  constexpr int RED = kWaves * RR * NA * 1024;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * BUF > RED ? 2 * BUF : RED];
  __shared__ int odd_row[16 * RT];             // rows with an infinity or a NaN
  f32x4(*red)[RR * NA][64] = (f32x4(*)[RR * NA][64])lds;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = wave & 3, half = wave >> 2;
  const int li = lane & 15, lg = lane >> 4;
  int rt0, cg;
  if (!tile_of(g, rt0, cg)) return;
  const int row0 = rt0 * 16 * RT;
  const int group0 = (cg * 2 + half) * U;      // this wave's first column group

  // rows of a chunk: thread -> (row tid/32 + 16 j, four floats)
  constexpr int NL = RT;
  int xm[NL], hm[NL], dn[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    xm[j] = hm[j] = min(row0 + 16 * j + (tid >> 5), g.M - 1);
    dn[j] = g.done[xm[j]];
  }
  state_rows(g, hm, dn);
  if (tid < 16 * RT) odd_row[tid] = 0;

  const size_t group_stride = (size_t)g.kn * PB * GB;
  const uint8_t* wbase = g.w + (size_t)group0 * group_stride;
  uint32_t woff[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    if (KIND == GRU && t < U)
      woff[t] = (uint32_t)(t * group_stride) + lane * 16;
    else if (KIND == LSTM)
      woff[t] = (uint32_t)((t >> 1) * group_stride) + (t & 1) * 1024 + lane * 16;
    else
      woff[t] = (uint32_t)((li >> 3) * group_stride) + 1024 + (lg * 8 + (li & 7)) * 16;
  }

  f32x4 acc[RT][NA];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int t = 0; t < NA; ++t) acc[r][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  const int nc = g.kn / KW, c1 = g.k1 / KW, c2 = g.k2 / KW;
  f32x4 a[NL];
  u32x4 b[2][PB][NB];
  auto load_b = [&](auto slotc, int c) __attribute__((always_inline)) {
    constexpr int SL = decltype(slotc)::value;
    const uint8_t* wp = wbase + (size_t)(min(c, nc - 1) * KW + kw) * (PB * GB);
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
      for (int t = 0; t < NB; ++t) b[SL][p][t] = *(const u32x4*)(wp + (woff[t] + p * GB));
  };
  // Where the next chunk to load has its rows.  Moved on ahead of an iteration's instructions, so
  // that these stay one block for the scheduler (selects around the loads become branches); it
  // stays on the last chunk.
  const uint8_t* from = (const uint8_t*)g.x1;
  uint32_t from_pitch = (uint32_t)g.I1 >> 5;
  int from_c = 0, from_state = 0;
  auto advance = [&]() __attribute__((always_inline)) {
    if (from_c + 1 >= nc) return;
    ++from_c;
    from += 512;
    if (from_c == c1) {
      from = (const uint8_t*)g.x2;
      from_pitch = (uint32_t)g.I2 >> 5;
    }
    if (from_c == c2) {
      from = (const uint8_t*)g.h_in;
      from_pitch = (uint32_t)g.S >> 5;
      from_state = 1;
    }
  };
  auto load_a = [&]() __attribute__((always_inline)) {
    const uint8_t* base = from + (tid & 31) * 16;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const uint32_t m = from_state ? hm[j] : xm[j];
      a[j] = *(const f32x4*)(base + ((size_t)(m * from_pitch) << 7));
    }
  };
  // Place of (row, K step of the chunk, lane group) in a term's 1 KB operand of (row tile, K step):
  // rows are exchanged by (lane group, K step), so that the lanes of a store, which differ in
  // these, spread over the banks.
  auto slot_of = [&](int row, int ks, int kg) { return 16 * kg + (row ^ ((kg << 2) | ks)); };
  float left[NL] = {};
  // piece j of this thread's rows of chunk c into buffer buf
  auto store_a = [&](int c, int buf, int j) __attribute__((always_inline)) {
    uint8_t* dst = lds + buf * BUF;
    const int ks = (tid & 31) >> 3, kg = (tid & 7) >> 1, hf = tid & 1;
    uint8_t* at = dst + ks * (NP * 1024) + slot_of(tid >> 5, ks, kg) * 16 + hf * 8 + j * KW * (NP * 1024);
    const unsigned keep = ((c >= c2) & (dn[j] != 0)) ? 0u : ~0u;
    u32x2 t[3];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      unsigned t0, t1, t2;
      float v0 = a[j][2 * p], v1 = a[j][2 * p + 1];
      v0 = __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v0) & keep);
      v1 = __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v1) & keep);
      split_pair(v0, v1, t0, t1, t2, left[j]);
      t[0][p] = t0;
      t[1][p] = t1;
      t[2][p] = t2;
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) *(u32x2*)(at + q * 1024) = t[q];
  };
  const int rd_slot = slot_of(li, kw, lg) * 16 + kw * (NP * 1024);
  // the products of row tile r of a chunk
  auto products = [&](auto slotc, int r) __attribute__((always_inline)) {
    constexpr int SL = decltype(slotc)::value;
    const uint8_t* src = lds + SL * BUF + rd_slot + r * KW * (NP * 1024);
    bf16x8 x[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) x[q] = *(const bf16x8*)(src + q * 1024);
    auto term = [&](int wq, int xq) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < NB; ++t)
        acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b[SL][wq][t]), x[xq], acc[r][t], 0, 0, 0);
    };
    term(2, 0);
    term(0, 2);
    term(1, 1);
    term(1, 0);
    term(0, 1);
    term(0, 0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  load_a();
  load_b(I0{}, 0);
#pragma unroll
  for (int j = 0; j < NL; ++j) store_a(0, 0, j);
  advance();
  load_a();
  load_b(I1{}, 1);  // (the order of the loop: the waits of its first trip are those of every trip)
  __syncthreads();
  // Iteration c: products of chunk c, rows of chunk c + 1 into the other buffer, loads of c + 2
  // (past the end: the last chunk again, unused; no conditions around the loads).  The two waves
  // of a SIMD leave the barrier together, so that each has to mix its own matrix and vector
  // instructions: in separate stretches both would use the one pipe, then both the other.
  auto iter = [&](auto slotc, int c) __attribute__((always_inline)) {
    constexpr int SL = decltype(slotc)::value;
    if (KIND == GRU && c == c2) {
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        acc[r][NA - 1] = acc[r][NA - 2];
        acc[r][NA - 2] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
    advance();
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      products(slotc, r);
      store_a(c + 1, SL ^ 1, r);
    }
    load_a();
    load_b(slotc, c + 2);
#pragma unroll
    for (int i = 0; i < RT * NB * 6; ++i) {  // one matrix instruction, two vector instructions
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
    }
    __syncthreads();
  };
  int c = 0;
  for (; c + 1 < nc; c += 2) {
    iter(I0{}, c);
    iter(I1{}, c + 1);
  }
  if (c < nc) iter(I0{}, c);

  // What the gates need, requested ahead of the exchange of sums.  Thread -> unit (half, four of
  // the half's sixteen, one of them), rows lane/4 + 16 j: a wave reads its sums from 64
  // neighbouring words of LDS.
  const int un = wave * 4 + (lane & 3), unit = cg * 32 + un, erow = lane >> 2;
  float bias[2][4] = {}, prev[RT];
  int gdn[RT], ghm[RT];
#pragma unroll
  for (int j = 0; j < RT; ++j) {
    ghm[j] = min(row0 + 16 * j + erow, g.M - 1);
    gdn[j] = g.done[ghm[j]];
  }
  state_rows(g, ghm, gdn);
#pragma unroll
  for (int j = 0; j < RT; ++j) prev[j] = g.h_in[(size_t)ghm[j] * g.S + (KIND == LSTM ? g.H : 0) + unit];
#pragma unroll
  for (int q = 0; q < (KIND == LSTM ? 4 : 3); ++q) {
    bias[0][q] = g.b1[q * g.H + unit];
    bias[1][q] = g.b2[q * g.H + unit];
  }
#pragma unroll
  for (int j = 0; j < NL; ++j)
    if (left[j] != left[j]) odd_row[16 * j + (tid >> 5)] = 1;

  // the four partial sums of a half, RR row tiles at a time, in wave order
#pragma unroll
  for (int rd = 0; rd < RT / RR; ++rd) {
    if (rd) __syncthreads();
#pragma unroll
    for (int r = 0; r < RR; ++r)
#pragma unroll
      for (int t = 0; t < NA; ++t) red[wave][r * NA + t][lane] = acc[rd * RR + r][t];
    __syncthreads();
    {
      const int hf = wave >> 2, eq = wave & 3, er = lane & 3;
      const int gq = eq >> 1, hq = eq & 1;
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        int tl[4], ln[4];
        if (KIND == LSTM) {
          tl[0] = tl[1] = 2 * gq;
          tl[2] = tl[3] = 2 * gq + 1;
          ln[0] = ln[2] = hq;
          ln[1] = ln[3] = 2 + hq;
        } else {
          tl[0] = tl[1] = gq;
          tl[2] = U + 1;
          tl[3] = U;
          ln[0] = hq;
          ln[1] = 2 + hq;
          ln[2] = ln[3] = eq;
        }
        float sum[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float* src = (const float*)&red[4 * hf][r * NA + tl[q]][16 * ln[q] + erow] + er;
          float v = src[0];
#pragma unroll
          for (int w = 1; w < 4; ++w) v += src[w * (RR * NA * 64 * 4)];
          sum[q] = v;
        }
        const int j = rd * RR + r, m = row0 + 16 * j + erow;
        if (m < g.M) {
          float* o = (float*)g.out + (size_t)m * g.S;
          const bool rs = gdn[j] != 0;
          bool odd = odd_row[16 * j + erow] != 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) odd |= !finite(sum[q]);
          if (__builtin_expect(odd, 0))
            plain_sums<KIND, XT, PB>(g, m, rs, unit, sum);
          const float before = rs ? 0.0f : prev[j];
          if (KIND == LSTM)
            cell_lstm(o, g.H, unit, sum, bias, before);
          else
            cell_gru(o, unit, sum, bias, before);
        }
      }
    }
  }
}

// Which block of tiles an XCD gets: of the divisions that give the XCDs the fewest rounds of workgroups
// the one whose block has the fewest bytes of rows and weights, which its L2 has to fetch.  (Rows or
// columns only, as before: FC 2304 -> 512 at 1024 rows 17.9, 19.5 against 17.1 us, GRU 512 at 1024 rows 24.8,
// 23.6 against 22.6.)
unsigned deal(DenseArgs& g, long long tile_row_bytes, long long group_bytes) {
  long long least = -1;
  for (int rows = 1; rows <= 8; rows *= 2) {
    const int per_rt = (g.n_rt + rows - 1) / rows, per_cg = (g.n_cg * rows + 7) / 8;
    const long long rounds = ((long long)per_rt * per_cg + 31) / 32;
    const long long cost = (rounds << 40) + per_rt * tile_row_bytes + per_cg * group_bytes;
    if (least >= 0 && cost >= least) continue;
    least = cost;
    g.xcd_rows = rows == 8 ? 3 : rows / 2;
    g.per_rt = per_rt;
    g.per_cg = per_cg;
  }
  g.rcp_cg = (uint32_t)((0x100000000ull + g.per_cg - 1) / g.per_cg);  // (exact: per_rt * per_cg^2 is far below 2^32)
  return 8u * g.per_rt * g.per_cg;
}

template <int KIND, int XT, int PB, int RT, int U, int DA, int DB, bool OUT16>
hipError_t launch_cfg(DenseArgs g, hipStream_t st) {
  g.n_rt = (g.M + 16 * RT - 1) / (16 * RT);
  g.n_cg = KIND == FC ? g.N / (16 * U) : g.H / (8 * U);
  const long long row_bytes = 16LL * RT * g.kn * 32 * (in_f32(XT) ? 4 : 2);
  const unsigned blocks = deal(g, row_bytes, (long long)U * g.kn * PB * group_bytes(KIND));
  if constexpr (KIND == FC && !OUT16)  // (features leave in bf16 only where there are no measurements)
    if (g.meas.B > 0) {
      g.blocks = (int)blocks;
      dense_split_kernel<KIND, XT, PB, RT, U, DA, DB, OUT16, true>
          <<<blocks + (g.meas.B + kMeasRows - 1) / kMeasRows, kThreads, 0, st>>>(g);
      return hipGetLastError();
    }
  dense_split_kernel<KIND, XT, PB, RT, U, DA, DB, OUT16, false><<<blocks, kThreads, 0, st>>>(g);
  return hipGetLastError();
}

template <int KIND, int RT>
hipError_t launch_tile_t(DenseArgs g, hipStream_t st) {
  g.n_rt = (g.M + 16 * RT - 1) / (16 * RT);
  g.n_cg = g.H / 32;
  const unsigned blocks = deal(g, 16LL * RT * g.kn * 128, 4LL * g.kn * 3 * group_bytes(KIND));
  cell_tile_kernel<KIND, RT><<<blocks, kThreads, 0, st>>>(g);
  return hipGetLastError();
}
template <int KIND>
hipError_t launch_tile(const DenseArgs& g, hipStream_t st) {
  // The smallest tile whose grid is one round of workgroups: what a workgroup takes grows with its rows.  512
  // units, us, 16 / 32 / 64 rows per workgroup: GRU, 256 rows 11.0 / 13.8 / 19.5, 512 rows 19.9 / 14.4 / 19.3, 768 rows 28.6 / 25.4 /
  // 20.0, 1024 rows 39 / 27 / 22.1, 1536 rows 58 / 39.6 / 39.8; LSTM, 256 rows 13.4 / 16.6 / 24.7, 512 rows 23.9 / 17.3 / 25.3, 1024
  // rows 47 / 33 / 27.3.
  auto one_round = [&](int rt) { return (long long)((g.M + 16 * rt - 1) / (16 * rt)) * (g.H / 32) <= 256; };
  if (one_round(1)) return launch_tile_t<KIND, 1>(g, st);
  if (one_round(2)) return launch_tile_t<KIND, 2>(g, st);
  return launch_tile_t<KIND, 4>(g, st);
}

long long split_workgroups(long long M, int n_col, int rt, int u) {
  return ((M + 16 * rt - 1) / (16 * rt)) * (n_col / u);
}

// Rows and columns per workgroup, in units of 16 rows x 16 outputs or 8 hidden units.  A round of
// workgroups (256, one per CU) takes about as long with one workgroup as with 256, the longer the
// larger the tile; a larger tile needs fewer bytes per product out of the L2, which is what bounds many
// rows.  So it is the smallest tile whose grid is one round.  Launch times (us, the launch's own 2.7 included):
//   FC 2304 -> 512, fp32     1 x 1   2 x 1   2 x 2   2 x 4   4 x 4
//          64 rows             6.2     8.4    10.0    14.6
//         256                 11.8    10.2    10.3    14.6    24.0
//         512                 24.0    16.0    10.8    14.9    24.4
//        1024                                 20.5    17.5    24.6
//        2048                                 34.7    32.0    27.4   (with the division by deal(); 39.3 before)
//   GRU 512 -> 512, fp32      1 x 1   2 x 1   2 x 2   2 x 4
//          64 rows             6.6     8.0     8.3    12.1
//         256                 21.2    16.6     9.4    12.1
//         333                                 15.2    12.2
//         512                                 17.3    12.9
//   LSTM 512 -> 512, fp32, 512 rows           21.3    15.5
//   FC 2304 -> 512, bf16: 600 rows 2 x 2 8.6, 2 x 4 6.8, 4 x 4 8.2; 2048 rows 15.8, 12.5, 10.9 (before 15.6)
//   FC 4608 -> 256, fp16: 512 rows 2 x 1 8.2, 2 x 2 6.9; 2048 rows 2 x 2 15.8, 2 x 4 13.1, 4 x 4 18.4 (15.9)
// Beyond one round of all of them the FC takes the one of 2 x 4 and 4 x 4 with the less time over its
// rounds, one of 4 x 4 counted as 1.6 (fp32 at 2600 rows 45.0, 48.5; at 4096 65, 56).  Weights in 16 bits leave room
// for two workgroups of 2 x 2 on a CU, one's loads behind the other's products: cells with one
// term stay with that (GRU 512 rows 9.3, 2 x 4 9.0; 1000 rows 16.2, 16.1).
// DA, DB by what fits the registers: all tiles but those with two workgroups per CU have 256, none spills
// but the LSTM's and GRU's of three terms would at 2 x 4 with two steps in flight.
// The bits of a result do not depend on any of this.
template <int KIND, int XT, int PB, bool OUT16>
hipError_t launch_kind(const DenseArgs& g, hipStream_t st) {
  const int n_col = KIND == FC ? g.N / 16 : g.H / 8;
  auto rounds = [&](int rt, int u) { return (split_workgroups(g.M, n_col, rt, u) + 255) / 256; };
  constexpr bool F32 = XT == X_F32;
  if (rounds(1, 1) <= 1) return launch_cfg<KIND, XT, PB, 1, 1, 4, 4, OUT16>(g, st);
  if constexpr (KIND != FC || F32)
    if (rounds(2, 1) <= 1) return launch_cfg<KIND, XT, PB, 2, 1, 3, 3, OUT16>(g, st);
  if constexpr (KIND == FC) {
    constexpr int D = F32 ? 1 : 2;
    if (rounds(2, 2) <= 1 || n_col % 4 != 0) return launch_cfg<KIND, XT, PB, 2, 2, D, D, OUT16>(g, st);
    if (rounds(2, 4) <= 1 || 5 * rounds(2, 4) < 8 * rounds(4, 4)) return launch_cfg<KIND, XT, PB, 2, 4, 2, D, OUT16>(g, st);
    return launch_cfg<KIND, XT, PB, 4, 4, 1, 1, OUT16>(g, st);
  } else if constexpr (PB == 3) {
    if (rounds(2, 2) <= 1) return launch_cfg<KIND, XT, PB, 2, 2, 2, 2, OUT16>(g, st);
    return launch_cfg<KIND, XT, PB, 2, 4, 1, 1, OUT16>(g, st);
  } else {
    return launch_cfg<KIND, XT, PB, 2, 2, 1, 1, OUT16>(g, st);
  }
}

// Packing runs at every weight update, 24 results per eight weights: two builds of the loops, the
// second with 256-bit vectors where the host has them.
#define SF_INLINE inline __attribute__((always_inline))
#if defined(__HIP_DEVICE_COMPILE__) || !defined(__x86_64__)
#define SF_AVX2
#else
#define SF_AVX2 __attribute__((target("avx2")))
#endif
bool host_avx2() {
#if defined(__HIP_DEVICE_COMPILE__) || !defined(__x86_64__)
  return false;
#else
  return __builtin_cpu_supports("avx2");
#endif
}

// Eight neighbouring weights -> one operand of a lane per term, `stride` elements apart.  bf16 to
// nearest, ties to even; what would become infinite is cut off.
SF_INLINE void put8(const float* src, int terms, bool f16, uint16_t* dst, size_t stride) {
  if (f16) {
    for (int e = 0; e < 8; ++e) dst[e] = conv_weight_bits(src[e], true);
    return;
  }
  typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
  typedef float f32x8 __attribute__((ext_vector_type(8)));
  typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
  f32x8 r;
  memcpy(&r, src, sizeof(r));
  for (int q = 0; q < terms; ++q) {
    const u32x8 u = __builtin_bit_cast(u32x8, r);
    const u32x8 up = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
    const u32x8 inf = (u32x8)((up & 0x7F800000u) == 0x7F800000u);  // all ones where true
    const u32x8 t = (up & ~inf) | (u & 0xFFFF0000u & inf);
    const u16x8 h = __builtin_convertvector(t >> 16, u16x8);
    memcpy(dst + q * stride, &h, sizeof(h));
    r -= __builtin_bit_cast(f32x8, t);
  }
}

SF_INLINE void pack_fc_loops(const float* w, int N, int K, int terms, bool f16, uint16_t* out) {
  const int kn = K / 32;
  for (int nb = 0; nb < N / 16; ++nb)
    for (int s = 0; s < kn; ++s)
      for (int lg = 0; lg < 4; ++lg)
        for (int i = 0; i < 16; ++i)
          put8(w + (size_t)(nb * 16 + i) * K + 32 * s + 8 * lg, terms, f16,
               out + (((size_t)nb * kn + s) * terms * 64 + lg * 16 + i) * 8, 64 * 8);
}
SF_INLINE void pack_cell_loops(const float* w_ih, const float* w_hh, int I, int H, int lstm, int terms, uint16_t* out) {
  const int kn = (I + H) / 32, G = lstm ? 4 : 3;
  const size_t gb = group_bytes(lstm ? LSTM : GRU) / 2;
  for (int gr = 0; gr < H / 8; ++gr)
    for (int s = 0; s < kn; ++s) {
      uint16_t* dst = out + ((size_t)gr * kn + s) * terms * gb;
      const float* src = 32 * s < I ? w_ih + 32 * s : w_hh + (32 * s - I);
      const size_t pitch = 32 * s < I ? I : H;
      for (int q = 0; q < G; ++q)
        for (int lg = 0; lg < 4; ++lg)
          for (int i = 0; i < 8; ++i) {
            const size_t slot = q < 2 || lstm ? (size_t)(q >> 1) * 64 + lg * 16 + (q & 1) * 8 + i : (size_t)64 + lg * 8 + i;
            put8(src + ((size_t)q * H + gr * 8 + i) * pitch + 8 * lg, terms, false, dst + slot * 8, gb);
          }
    }
}
void pack_fc_plain(const float* w, int N, int K, int terms, bool f16, uint16_t* out) { pack_fc_loops(w, N, K, terms, f16, out); }
SF_AVX2 void pack_fc_avx2(const float* w, int N, int K, int terms, bool f16, uint16_t* out) {
  pack_fc_loops(w, N, K, terms, f16, out);
}
void pack_cell_plain(const float* w_ih, const float* w_hh, int I, int H, int lstm, int terms, uint16_t* out) {
  pack_cell_loops(w_ih, w_hh, I, H, lstm, terms, out);
}
SF_AVX2 void pack_cell_avx2(const float* w_ih, const float* w_hh, int I, int H, int lstm, int terms, uint16_t* out) {
  pack_cell_loops(w_ih, w_hh, I, H, lstm, terms, out);
}

}  // namespace

// FC: N outputs from K inputs, whole column groups and whole K steps.
bool dense_fc_supported(int K, int N) { return K > 0 && (K % 32) == 0 && N > 0 && (N % 32) == 0; }
bool dense_cell_supported(int I1, int I2, int H) {
  return I1 > 0 && (I1 % 32) == 0 && (I2 % 32) == 0 && H > 0 && (H % 32) == 0;
}
// FC layer on 16-bit rows: up to two rounds of the largest tile; beyond, k_fc16.hip.  Whole steps, this kernel
// against that one: bf16, 16 rows 24 against 29 us, 256 rows 32, 36, 2048 rows 95, 91; fp16 4608 -> 256, 101 rows
// 83, 94, 1024 rows 253, 259, 2048 rows 477, 477, 4096 rows 870, 863.  (A handle keeps one of the two, and
// a handle for 2048 rows also takes calls of few.)
bool dense_fc_small(int M, int N) { return split_workgroups(M, N / 16, 4, 2) <= 512; }
// Cells: up to two rounds of the 32-row tile.  Beyond, cell_tile_kernel in fp32 (GRU 512 -> 512, us: 256
// rows 9.7 against 11.0, 512 rows 13.4, 14.4, 768 rows 23.4, 20, 1024 rows 25.2, 22.1, 2048 rows 48, 42.5) and k_rnn_bf16.hip in bf16 (at 512 rows 10
// against 20 us, at 1024 rows 24 against 21; 256 -> 256 at 1000 rows 8 against 14).  The kernels'
// sums run in different orders (and the state enters k_rnn_bf16.hip in two terms), so that this is
// settled once, by the largest batch.
bool dense_cell_small(int M, int H) { return split_workgroups(M, H / 8, 2, 2) <= 512; }
bool dense_cell_tile_supported(int I1, int I2, int H) {
  return I1 > 0 && (I1 % 128) == 0 && (I2 % 128) == 0 && H > 0 && (H % 128) == 0;
}

// w [N][K] -> [N / 16][K / 32][terms][64][8]; terms: 3 (fp32 weights) or 1 (bf16, or fp16 if f16).
size_t dense_fc_pack_size(int N, int K, int terms) { return (size_t)N * K * terms; }
void dense_pack_fc(const float* w, int N, int K, int terms, bool f16, uint16_t* out) {
  (host_avx2() ? pack_fc_avx2 : pack_fc_plain)(w, N, K, terms, f16, out);
}

// w_ih [G*H][I], w_hh [G*H][H] -> [H / 8][(I + H) / 32][terms][operands of a group]: tile columns
// [i f | g o] (LSTM) or [r z] and the eight n columns of every lane group (GRU).
size_t dense_cell_pack_size(int I, int H, int lstm, int terms) {
  return (size_t)(H / 8) * ((I + H) / 32) * terms * (group_bytes(lstm ? LSTM : GRU) / 2);
}
void dense_pack_cell(const float* w_ih, const float* w_hh, int I, int H, int lstm, int terms, uint16_t* out) {
  (host_avx2() ? pack_cell_avx2 : pack_cell_plain)(w_ih, w_hh, I, H, lstm, terms, out);
}

// The smallest tile's LDS has to hold the rows of a workgroup.
static_assert(kMeasThreads == kThreads, "workgroups of the FC layer's launch");
bool dense_fc_takes_meas(int n0, int n1) { return meas_lds(n0, n1) <= kWaves * 16 * 36; }

// meas: measurement layers to be computed by further workgroups of the launch, or null: their time passes
// beside the FC layer's (as a launch of their own 6.4 us at 333 rows, latency for the most part).
// x [M][K] (x_type 0 fp32, 1 bf16, 2 fp16), w packed with three terms for fp32 rows and one for
// 16-bit rows; out [M][N] = relu(x w^T + bias), fp32 or (out_bf16) bf16.
hipError_t launch_dense_fc(const void* x, int x_type, const uint16_t* w, const float* bias, void* out, int out_bf16,
                           int M, int K, int N, const MeasArgs* meas, hipStream_t st) {
  if (M == 0) return hipSuccess;
  if (!dense_fc_supported(K, N) || (meas && (out_bf16 || !dense_fc_takes_meas(meas->n0, meas->n1)))) return hipErrorInvalidValue;
  DenseArgs g{};
  if (meas) g.meas = *meas;
  g.x1 = x; g.w = (const uint8_t*)w; g.b1 = bias; g.out = out;
  g.M = M; g.I1 = K; g.N = N; g.k1 = g.k2 = g.kn = K / 32;
  if (x_type == X_F32) return out_bf16 ? hipErrorInvalidValue : launch_kind<FC, X_F32, 3, false>(g, st);
  if (x_type == X_BF16)
    return out_bf16 ? launch_kind<FC, X_BF16, 1, true>(g, st) : launch_kind<FC, X_BF16, 1, false>(g, st);
  return out_bf16 ? hipErrorInvalidValue : launch_kind<FC, X_F16, 1, false>(g, st);
}

// terms: of the packed weights (3 or 1); x_type: features in fp32 (0), or with one term: x1 in bf16
// (1), fp32 features to be rounded to bf16 (2); tile: cell_tile_kernel.
hipError_t launch_dense_cell(int lstm, int B, int I1, int I2, int H, const void* x1, int x_type, const float* x2,
                             const float* h_in, const uint8_t* done, const uint16_t* w, int terms, const float* b_ih,
                             const float* b_hh, float* h_out, const int32_t* ids, int n_env, int tile, hipStream_t st) {
  if (B == 0) return hipSuccess;
  if (!x2) I2 = 0;
  if (!dense_cell_supported(I1, I2, H) || (x_type && terms != 1) || (x_type == 1 && I2)) return hipErrorInvalidValue;
  DenseArgs g{};
  g.x1 = x1; g.x2 = x2; g.h_in = h_in; g.done = done; g.ids = ids; g.w = (const uint8_t*)w;
  g.b1 = b_ih; g.b2 = b_hh; g.out = h_out;
  g.M = B; g.I1 = I1; g.I2 = I2; g.H = H; g.S = lstm ? 2 * H : H; g.n_env = n_env;
  g.k1 = I1 / 32; g.k2 = (I1 + I2) / 32; g.kn = g.k2 + H / 32;
  if (tile) {
    if (terms != 3 || !dense_cell_tile_supported(I1, I2, H)) return hipErrorInvalidValue;
    return lstm ? launch_tile<LSTM>(g, st) : launch_tile<GRU>(g, st);
  }
  if (terms == 3) return lstm ? launch_kind<LSTM, X_F32, 3, false>(g, st) : launch_kind<GRU, X_F32, 3, false>(g, st);
  if (x_type == 1) return lstm ? launch_kind<LSTM, X_BF16, 1, false>(g, st) : launch_kind<GRU, X_BF16, 1, false>(g, st);
  if (x_type == 2) return lstm ? launch_kind<LSTM, X_ROUND, 1, false>(g, st) : launch_kind<GRU, X_ROUND, 1, false>(g, st);
  return lstm ? launch_kind<LSTM, X_F32, 1, false>(g, st) : launch_kind<GRU, X_F32, 1, false>(g, st);
}

}  // namespace sf
