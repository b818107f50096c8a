// The recurrent core over all T steps of N trajectories in one launch (paper, Sec. 3.1: the learner
// recomputes the network on the trajectories it was sent), weights resident in registers.
//
// As one launch per step (k_dense_split.hip on N rows) a step pays a launch, 50 MB of weights out of
// the L2s (every row tile reads them again) and the latency of its operands: 7.2 us for an LSTM 512 ->
// 512 in fp32 on 64 rows, 4.9 for a GRU 256 -> 256 in bf16.  Here a workgroup keeps the weights of eight
// hidden units (eight waves, an eighth of K each: up to 120 registers) and takes 16 RT trajectories
// through all steps; what the workgroups of a row tile exchange per step is the new state, 2 KB per row.
// Arithmetic, split of the operands into bf16 terms and gates are those of k_dense_split.hip; the order of
// the sums is this kernel's own: per wave its part of the features, then its part of the state.
//
// Exchange.  The states go to h_seq, where they have to go anyway.  A launch ahead of this one fills that
// array's h columns with a bit pattern that no state has (a NaN whose bits are all ones); a state is stored
// with device scope and read by the other workgroups with device-scope loads, which go past the caches
// that are not coherent across the XCDs, until the pattern is gone.  Each word is its own flag: no
// counters, no fences, no cache write-back, one store and one load of latency per step.  The bytes read
// count (every workgroup of a row tile reads all its states from the memory side, 1 MB per XCD and step):
// exchanged in three bf16 terms, 1.5 times as much, a step took twice as long.  So does the size of a
// store: eight units of a row, 32 bytes, by one wave (16 bytes: 1.6 times as long; the memory has to merge
// them).  The features' products of a step run while its states travel.
//
// Progress.  A workgroup takes its row tile and its units by a ticket when it starts to run, so that the
// row tiles are filled one after the other and a running workgroup waits only for workgroups that run
// or are next to.  A wait ends after `limit` reads whatever happens: then the trajectories of that row tile
// are marked and its workgroups leave; the other tiles do not notice.
//
// What the terms cannot compute: the products of an infinity, a NaN or of numbers whose product overflows do
// not add up to the product.  Such a sum is not finite; its trajectory, whose row is a column of the matrix
// instructions of its own, is marked and goes on (a NaN of other bits than the pattern), and so does every
// other one, with the same bits as without it.
//
// core_seq_plain_kernel, launched behind this one, computes the marked trajectories again, in plain fp32 and
// without an exchange between workgroups: from the first such step to the episode's end behind the last one,
// or all steps of a tile that was given up (the other trajectories' workgroups return at once).
#include <type_traits>

#include "sf_cell.h"
#include "sf_exchange.h"
#include "sf_internal.h"
#include "sf_split.h"

namespace sf {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kPlain = 1024;  // threads of core_seq_plain_kernel
constexpr int kMaxX = 3 * 32 * kWaves, kMaxH = 2 * 32 * kWaves;  // see core_seq_supported

struct SeqArgs {
  DenseArgs d;    // x1, x2, w, b1, b2, I1, I2, H, S, k1, k2, kn; M = N trajectories
  const float* h0;       // [N][S]
  const uint8_t* done;   // [T][N]
  float* seq;            // [T][N][S]
  int T, n_cg;
  int limit;             // reads of a word that has not come (negative: every tile is given up at once)
  unsigned* ticket;
  unsigned* mark;        // [N][2], see kNone
};
// A trajectory's marks: the first step with a sum that is not finite, plus one (0: its row tile was given
// up; kNone: neither), and the last such step.
constexpr unsigned kNone = 0xFFFFFFFFu;

// also sets the n_words words of the ticket and the marks
__global__ __launch_bounds__(256) void core_seq_fill_kernel(float* seq, long long rows, int H, int S, unsigned* words, int n_words) {
  const int per = H / 4;
  const long long n = rows * per;
  for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < n_words; i += (int)(256 * gridDim.x))
    words[i] = i & 1 ? kNone : 0;
  const u32x4 v = {kNotYet, kNotYet, kNotYet, kNotYet};
  for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += 256ll * gridDim.x)
    *(u32x4*)(seq + i / per * S + 4 * (i % per)) = v;
}

// KX, KH: K steps (of 32) of a wave over the features / over the state; RT: row tiles of 16.
template <int KIND, int XT, int PB, int RT, int KX, int KH>
__global__ __launch_bounds__(kThreads, 2) void core_seq_kernel(SeqArgs g) {
  constexpr int GB = group_bytes(KIND), NB = 2, NA = KIND == GRU ? 3 : 2;
  constexpr int P32 = 36, P16 = 20;  // pitch of a row in LDS (floats): 16-byte accesses without conflicts
  constexpr int ROWS = 16 * RT;
  constexpr int NX = XT == X_F32 ? 2 * RT : RT;  // feature loads per K step
  constexpr int NH = 2 * RT;                     // state loads per K step
  __shared__ __attribute__((aligned(16))) float corner[kWaves][ROWS * P32];
  // partial sums; groups of 16 lanes 8 words apart modulo 64, so that the gates read different banks
  constexpr int TILE = 4 * 72;                   // floats
  __shared__ __attribute__((aligned(16))) float red[2][kWaves][RT * NA][TILE];
  __shared__ unsigned first_word;
  __shared__ int lost[2];                        // a wait was given up, by step (a wave may be one step ahead)
  __shared__ int odd[2][ROWS];                   // first (plus one) and last step of a row with a sum that is not finite

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int M = g.d.M, H = g.d.H, S = g.d.S;
  if (tid == 0) {
    first_word = __hip_atomic_fetch_add(g.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    lost[0] = lost[1] = 0;
  }
  if (tid < ROWS) odd[0][tid] = odd[1][tid] = 0;
  __syncthreads();
  const int ticket = __builtin_amdgcn_readfirstlane((int)first_word);
  const int row0 = ticket / g.n_cg * ROWS, cg = ticket % g.n_cg;

  // ---- weights of the wave's K steps ----
  uint32_t woff[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t)  // (GRU: the eight n columns twice)
    woff[t] = KIND == LSTM || t == 0 ? t * 1024 + lane * 16 : 1024 + (lg * 8 + (li & 7)) * 16;
  const uint8_t* wbase = g.d.w + (size_t)cg * g.d.kn * PB * GB;
  const int kx0 = wave * KX, kh0 = g.d.k2 + wave * KH;
  u32x4 wx[KX][PB][NB], wh[KH][PB][NB];
  auto load_w = [&](u32x4 (&w)[PB][NB], int s) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
      for (int t = 0; t < NB; ++t) w[p][t] = *(const u32x4*)(wbase + ((size_t)s * PB + p) * GB + woff[t]);
  };
#pragma unroll
  for (int i = 0; i < KX; ++i) load_w(wx[i], min(kx0 + i, g.d.k2 - 1));
#pragma unroll
  for (int i = 0; i < KH; ++i) load_w(wh[i], min(kh0 + i, g.d.kn - 1));

  // ---- the gates: thread -> (row, unit, gate), the gates of a unit in neighbouring lanes ----
  // (a row's eight units in neighbouring lanes: 32 bytes per store; stored by 16 the memory behind the
  // caches has to merge them)
  const int q = tid & 3, er = (tid >> 2) & 3, eq = (tid >> 4) & 1, erow = tid >> 5;
  const int unit = cg * 8 + eq * 4 + er;
  // GRU: r, z, the features' and the state's part of n; LSTM: i, f, g, o
  const int tile = KIND == LSTM ? q >> 1 : q < 2 ? 0 : 4 - q;
  const int from = tile * TILE + 72 * (eq + (KIND == LSTM || q < 2 ? 2 * (q & 1) : 0)) + 4 * erow + er;
  float bias;
  if (KIND == LSTM || q < 2)
    bias = g.d.b1[q * H + unit] + g.d.b2[q * H + unit];
  else
    bias = (q == 2 ? g.d.b1 : g.d.b2)[2 * H + unit];
  float prev[RT];  // the unit's h (GRU) or c
#pragma unroll
  for (int r = 0; r < RT; ++r)
    prev[r] = g.h0[(size_t)min(row0 + 16 * r + erow, M - 1) * S + (KIND == LSTM ? H : 0) + unit];

  // ---- a step's features, one step ahead ----
  // (neighbouring lanes on neighbouring bytes, turned into operand order in an LDS corner of the wave's
  // own; past the last row: that row again, never stored)
  uint32_t xrow[NX], hoff[NH];
#pragma unroll
  for (int j = 0; j < NX; ++j) xrow[j] = min(row0 + (XT == X_F32 ? 8 * j + (lane >> 3) : 16 * j + (lane >> 2)), M - 1);
#pragma unroll
  for (int j = 0; j < NH; ++j) hoff[j] = 4u * ((uint32_t)min(row0 + 8 * j + (lane >> 3), M - 1) * S + (lane & 7) * 4);
  f32x4 xa[KX][NX];
  auto load_x = [&](int t) __attribute__((always_inline)) {
    const size_t r0 = (size_t)t * M;
#pragma unroll
    for (int i = 0; i < KX; ++i) {
      const int s = min(kx0 + i, g.d.k2 - 1);
      if constexpr (XT == X_F32) {
        const bool one = s < g.d.k1;
        const uint32_t pitch = one ? g.d.I1 : g.d.I2;
        const uint8_t* base = (const uint8_t*)((one ? (const float*)g.d.x1 + 32 * s : g.d.x2 + 32 * (s - g.d.k1)) + r0 * pitch);
#pragma unroll
        for (int j = 0; j < NX; ++j) xa[i][j] = *(const f32x4*)(base + 4u * (xrow[j] * pitch + (lane & 7) * 4));
      } else {
        const uint8_t* base = (const uint8_t*)((const uint16_t*)g.d.x1 + 32 * s + r0 * g.d.I1);
#pragma unroll
        for (int j = 0; j < NX; ++j) xa[i][j] = *(const f32x4*)(base + 2u * (xrow[j] * g.d.I1 + (lane & 3) * 8));
      }
    }
  };
  load_x(0);

  f32x4 acc[RT][NA];
  float left = 0.0f;  // (of the splitting: not needed, an infinity or a NaN shows in the sums)
  float* turn = corner[wave];
  auto mfma = [&](const u32x4& w, const u32x4& x, f32x4& c) __attribute__((always_inline)) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
  };
  // the products of a K step on a row tile; tile 1's accumulator: `second`
  auto terms = [&](auto f32c, const u32x4 (&w)[PB][NB], const u32x4* x, int r, int second) __attribute__((always_inline)) {
    constexpr bool F32 = decltype(f32c)::value;
    auto term = [&](int wq, int xq) __attribute__((always_inline)) {
      mfma(w[wq][0], x[xq], acc[r][0]);
      mfma(w[wq][1], x[xq], acc[r][second]);
    };
    // smallest products first
    if constexpr (F32 && PB == 3) {
      term(2, 0);
      term(0, 2);
      term(1, 1);
      term(1, 0);
      term(0, 1);
    } else if constexpr (F32) {
      term(0, 2);
      term(0, 1);
    }
    term(0, 0);
  };
  // ... of features, whose rows are in the corner
  auto products = [&](auto f32c, const u32x4 (&w)[PB][NB], int second) __attribute__((always_inline)) {
    constexpr bool F32 = decltype(f32c)::value;
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      u32x4 x[3];
      if constexpr (F32) {
        const f32x4 v0 = *(const f32x4*)(turn + (16 * r + li) * P32 + lg * 8);
        const f32x4 v1 = *(const f32x4*)(turn + (16 * r + li) * P32 + lg * 8 + 4);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          unsigned t0, t1, t2;
          split_pair(p < 2 ? v0[2 * p] : v1[2 * p - 4], p < 2 ? v0[2 * p + 1] : v1[2 * p - 3], t0, t1, t2, left);
          x[0][p] = t0;
          x[1][p] = t1;
          x[2][p] = t2;
        }
      } else {
        x[0] = __builtin_bit_cast(u32x4, *(const f32x4*)(turn + (16 * r + li) * P16 + lg * 4));
      }
      terms(f32c, w, x, r, second);
    }
  };

  for (int t = 0; t < g.T; ++t) {
    // ---- the features' products, while the states of the step before travel ----
    const uint8_t flag = g.done[(size_t)t * M + min(row0 + (lane & 31), M - 1)];
    const auto state = __builtin_amdgcn_make_buffer_rsrc((void*)(t == 0 ? g.h0 : g.seq + (size_t)(t - 1) * M * S), 0, 4 * M * S, 0x00027000);
    u32x4 hv[KH][NH];
    auto load_h = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < KH; ++i)
#pragma unroll
        for (int j = 0; j < NH; ++j)
          hv[i][j] = __builtin_amdgcn_raw_buffer_load_b128(state, hoff[j], 128 * (min(kh0 + i, g.d.kn - 1) - g.d.k2), kDeviceScope);
    };
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
      for (int n = 0; n < NA; ++n) acc[r][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int i = 0; i < KX; ++i) {
      if (kx0 + i >= g.d.k2) break;
#pragma unroll
      for (int j = 0; j < NX; ++j) {
        if constexpr (XT == X_F32)
          *(f32x4*)(turn + (8 * j + (lane >> 3)) * P32 + (lane & 7) * 4) = xa[i][j];
        else
          *(f32x4*)(turn + (16 * j + (lane >> 2)) * P16 + (lane & 3) * 4) = xa[i][j];
      }
      products(std::integral_constant<bool, XT == X_F32>{}, wx[i], KIND == GRU ? 2 : 1);
    }
    // ---- the states (asked for any earlier most have not come, and the reads that have to be repeated
    // hold up the stores: 147 against 116 us for 32 steps of an LSTM 512 on 64 rows) ----
    load_h();
    bool quit = false;
    for (int tries = 0; t > 0; ++tries) {
      unsigned missing = 0;
#pragma unroll
      for (int i = 0; i < KH; ++i)
#pragma unroll
        for (int j = 0; j < NH; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) missing |= (unsigned)(hv[i][j][e] == kNotYet);
      if (__all(missing == 0) && g.limit >= 0) break;
      quit = tries >= g.limit || ((tries & 63) == 63 && load_word(g.mark + 2 * row0) == 0);
      if (quit) break;
      load_h();
    }
    const unsigned reset = (unsigned)__ballot(flag != 0);  // by row
    load_x(min(t + 1, g.T - 1));
#pragma unroll
    for (int i = 0; i < KH; ++i) {
      if (kh0 + i >= g.d.kn) break;
#pragma unroll
      for (int j = 0; j < NH; ++j) {
        const unsigned keep = (reset >> (8 * j + (lane >> 3)) & 1) - 1;
        u32x4 v = hv[i][j];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] &= keep;
        *(u32x4*)(turn + (8 * j + (lane >> 3)) * P32 + (lane & 7) * 4) = v;
      }
      products(std::true_type{}, wh[i], 1);
    }
#pragma unroll
    for (int r = 0; r < RT; ++r) {
#pragma unroll
      for (int n = 0; n < NA; ++n) *(f32x4*)&red[t & 1][wave][r * NA + n][4 * lane + 8 * lg] = acc[r][n];
    }
    if (quit) lost[t & 1] = 1;
    __syncthreads();
    if (__builtin_expect(lost[t & 1] != 0, 0)) {  // (the same for all threads)
      if (tid < min(ROWS, M - row0))
        __hip_atomic_fetch_min(g.mark + 2 * (row0 + tid), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    // ---- the eight partial sums in wave order, gates, new state ----
    // (the other half of `red` is the next step's: one barrier per step)
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const float* src = &red[t & 1][0][r * NA][0] + from;
      float v = src[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += src[w * (RT * NA * TILE)];
      v += bias;
      const int m = row0 + 16 * r + erow;
      const float before = reset >> (16 * r + erow) & 1 ? 0.0f : prev[r];
      auto gate = [&](float a, auto k) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value * 0x55;  // the quad's lane k
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, a), K, 0xF, 0xF, true));
      };
      using Q0 = std::integral_constant<int, 0>;
      using Q1 = std::integral_constant<int, 1>;
      using Q2 = std::integral_constant<int, 2>;
      using Q3 = std::integral_constant<int, 3>;
      float h;
      if (KIND == LSTM) {
        const float a = q == 2 ? tanh_acc(v) : sigmoid_acc(v);
        prev[r] = gate(a, Q1{}) * before + gate(a, Q0{}) * gate(a, Q2{});
        h = gate(a, Q3{}) * tanh_acc(prev[r]);
      } else {
        const float a = sigmoid_acc(v), z = gate(a, Q1{});
        const float n = tanh_acc(gate(v, Q2{}) + gate(a, Q0{}) * gate(v, Q3{}));
        h = prev[r] = (1.0f - z) * n + z * before;
      }
      float* o = g.seq + ((size_t)t * M + m) * S + unit;
      if (m < M) {
        if (q == 0) __hip_atomic_store(o, h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (KIND == LSTM && q == 1) o[H] = prev[r];
      }
      // a sum with an infinity or a NaN in it, or of terms that overflow (behind the store, which the others
      // wait for: a NaN is stored again, with bits that no one waits for)
      if (__builtin_expect(!finite(v) || h != h, 0)) {
        if (odd[0][16 * r + erow] == 0) odd[0][16 * r + erow] = t + 1;  // (a row's threads are in one wave)
        odd[1][16 * r + erow] = t;
        if (h != h && q == 0 && m < M) __hip_atomic_store(o, __builtin_nanf(""), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  __syncthreads();
  if (tid < min(ROWS, M - row0) && odd[0][tid] != 0) {
    unsigned* at = g.mark + 2 * (row0 + tid);
    __hip_atomic_fetch_min(at, (unsigned)odd[0][tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(at + 1, (unsigned)odd[1][tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The marked trajectories without an exchange: a workgroup each, its state in LDS; a wave takes eight units, a
// lane one of them and every eighth run of eight numbers of K (eight lanes' weights are one cache line).  Whole
// passes on 64 trajectories of 32 steps, one of them never finite: LSTM 512 -> 512 4.2 ms, GRU 512 -> 512 3.4, in
// bf16 1.5 (a launch per step, where k_dense_split.hip computes such a row by a lane per unit: 23.3, 18.5, 17.4);
// all of them given up: 3.9, 3.0, 1.4.
template <int KIND, int XT, int PB>
__global__ __launch_bounds__(kPlain) void core_seq_plain_kernel(SeqArgs g) {
  constexpr int GB = group_bytes(KIND), NG = KIND == LSTM ? 4 : 3;
  __shared__ __attribute__((aligned(16))) float x[kMaxX], hs[2][kMaxH], cs[kMaxH];
  const int m = blockIdx.x, M = g.d.M, H = g.d.H, S = g.d.S, k1 = g.d.k1, k2 = g.d.k2, kn = g.d.kn;
  const unsigned first = load_word(g.mark + 2 * m);
  if (first == kNone) return;
  const int t0 = first == 0 ? 0 : (int)first - 1, last = first == 0 ? g.T : (int)load_word(g.mark + 2 * m + 1);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* before = t0 == 0 ? g.h0 + (size_t)m * S : g.seq + ((size_t)(t0 - 1) * M + m) * S;
  for (int n = tid; n < H; n += kPlain) {
    hs[t0 & 1][n] = before[n];
    cs[n] = KIND == LSTM ? before[H + n] : 0.0f;
  }
  for (int t = t0; t < g.T; ++t) {
    const size_t row = (size_t)t * M + m;
    const bool reset = g.done[row] != 0;
    if (reset && t > last) return;  // (nothing before this step matters to those behind it)
    for (int k = tid; k < 32 * k2; k += kPlain) {
      if constexpr (XT == X_F32)
        x[k] = k < 32 * k1 ? ((const float*)g.d.x1)[row * g.d.I1 + k] : g.d.x2[row * g.d.I2 + (k - 32 * k1)];
      else
        x[k] = __builtin_bit_cast(float, (unsigned)((const uint16_t*)g.d.x1)[row * g.d.I1 + k] << 16);
    }
    __syncthreads();  // (the states of the step before, too)
    float* const next = hs[(t + 1) & 1];
    for (int cg = wave; cg < H / 8; cg += kPlain / 64) {
      const int unit = 8 * cg + (lane & 7);
      // GRU: r, z, the features' and the state's part of n; LSTM: i, f, g, o
      float sum[4] = {};
      const uint8_t* group = g.d.w + (size_t)cg * kn * PB * GB;
      for (int i = lane >> 3; i < 4 * kn; i += 8) {
        const int s = i >> 2, lg = i & 3;
        const bool state = s >= k2;
        const float* from = state ? hs[t & 1] + 8 * i - 32 * k2 : x + 8 * i;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = state && reset ? 0.0f : from[e];
#pragma unroll
        for (int q = 0; q < NG; ++q) {
          const int slot = KIND == LSTM || q < 2 ? (q >> 1) * 64 + lg * 16 + (q & 1) * 8 + (lane & 7) : 64 + lg * 8 + (lane & 7);
          u32x4 w[PB];
#pragma unroll
          for (int p = 0; p < PB; ++p) w[p] = *(const u32x4*)(group + ((size_t)s * PB + p) * GB + slot * 16);
          float a = 0.0f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float we = 0.0f;
#pragma unroll
            for (int p = PB - 1; p >= 0; --p)
              we += __builtin_bit_cast(float, e & 1 ? w[p][e / 2] & 0xFFFF0000u : w[p][e / 2] << 16);
            a = fmaf(v[e], we, a);
          }
          if (KIND == GRU && q == 2)
            sum[state ? 3 : 2] += a;
          else
            sum[q] += a;
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int d = 8; d < 64; d *= 2) sum[q] += __shfl_xor(sum[q], d);
      float bias[2][4] = {};
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        bias[0][q] = g.d.b1[q * H + unit];
        bias[1][q] = g.d.b2[q * H + unit];
      }
      float* o = g.seq + row * S;
      float h, cell = 0.0f;
      if (KIND == LSTM)
        h = lstm_gates(sum, bias, reset ? 0.0f : cs[unit], cell);
      else
        h = gru_gates(sum, bias, reset ? 0.0f : hs[t & 1][unit]);
      if (lane < 8) {
        next[unit] = o[unit] = h;
        if (KIND == LSTM) cs[unit] = o[H + unit] = cell;
      }
    }
    __syncthreads();  // the features are used up
  }
}

template <int KIND, int XT, int PB, int RT, int KX, int KH>
hipError_t launch_rt(const SeqArgs& g, hipStream_t st) {
  const int blocks = (g.d.M + 16 * RT - 1) / (16 * RT) * g.n_cg;
  core_seq_kernel<KIND, XT, PB, RT, KX, KH><<<blocks, kThreads, 0, st>>>(g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  core_seq_plain_kernel<KIND, XT, PB><<<g.d.M, kPlain, 0, st>>>(g);
  return hipGetLastError();
}
template <int KIND, int XT, int PB, int KX, int KH>
hipError_t launch_k(const SeqArgs& g, int cus, hipStream_t st) {
  if constexpr (KX <= 2)  // (more leave no registers for a second row tile)
    if ((g.d.M + 15) / 16 * g.n_cg > cus) return launch_rt<KIND, XT, PB, 2, KX, KH>(g, st);
  return launch_rt<KIND, XT, PB, 1, KX, KH>(g, st);
}
template <int KIND, int XT, int PB>
hipError_t launch_kind(const SeqArgs& g, int cus, hipStream_t st) {
  const int kx = (g.d.k2 + kWaves - 1) / kWaves, kh = (g.d.kn - g.d.k2 + kWaves - 1) / kWaves;
  if (kx <= 1 && kh <= 1) return launch_k<KIND, XT, PB, 1, 1>(g, cus, st);
  if (kx <= 2 && kh <= 2) return launch_k<KIND, XT, PB, 2, 2>(g, cus, st);
  if constexpr (XT == X_F32)
    if (kx <= 3 && kh <= 2) return launch_k<KIND, XT, PB, 3, 2>(g, cus, st);
  return hipErrorInvalidValue;
}

}  // namespace

// Which passes run here.  Features and states of whole K steps, as many as a wave's registers hold the
// weights of; as many compute units as a row tile has workgroups (they wait for one another, and a unit holds
// one); rows whose workgroups run at once, 16 or 32 rows each (on 256 units 128 rows of 512), with three K steps of
// features per wave, which leave no room for a second row tile, two rounds of 16.  Whole passes, 32 x 64 and
// 32 x 120 / 8 x 256 samples, against a launch per step: GRU 512 342 -> 238, 550 -> 392 / 222 -> 235 us; with 128
// measurement features 393 -> 259, 600 -> 457 / 240 -> 271; in bf16 226 -> 172, 320 -> 247 / 129 -> 151; GRU 256 in
// bf16 656 -> 569, 1048 -> 961 / 548 -> 532, 8 x 512 995 -> 1006.
// And steps enough: the launches ahead and behind and the weights' way into registers take 9 us and more, a step
// saves 1.5 to 5.  From 16 to 256 rows of 32 to 512 units, both cells, both types: in one row tile 4 steps
// are faster everywhere (45.9 against 50.6 us to 54.1 against 61.7); beyond, 4 are not (LSTM 512 on 32 rows 72.1 against
// 64.8, GRU 256 on 128 rows 111.8 against 107.7), 5 with up to 256 units are (211.7 against 212.6 to 53.7
// against 64.2) and with 512 not (82.1 against 79.7 on 48 rows in bf16), 6 are (106.6 against 114.4 on 64).
// cus: compute units that the stream's workgroups may use.
bool core_seq_supported(int T, int N, int I1, int I2, int H, int x_type, int cus) {
  if (I1 <= 0 || I1 % 32 || I2 % 32 || H <= 0 || H % 32 || (x_type == 1 && I2)) return false;
  const int kx = ((I1 + I2) / 32 + kWaves - 1) / kWaves, kh = (H / 32 + kWaves - 1) / kWaves;
  if (kx > (x_type == 1 ? 2 : 3) || kh > 2) return false;
  const long long tiles = (N + 15) / 16;
  if (H / 8 > cus || T < (tiles == 1 ? 4 : H <= 256 ? 5 : 6)) return false;
  return (kx <= 2 ? (tiles + 1) / 2 * (H / 8) : (tiles * (H / 8) + 1) / 2) <= cus;
}

hipError_t launch_core_seq(int lstm, int T, int N, int I1, int I2, int H, const void* x1, int x_type, const float* x2,
                           const float* h0, const uint8_t* done, const uint16_t* w, int terms, const float* b_ih,
                           const float* b_hh, float* h_seq, unsigned* words, int limit, int cus, hipStream_t st) {
  if (!x2) I2 = 0;
  if (!core_seq_supported(T, N, I1, I2, H, x_type, cus) || (x_type != 0 && x_type != 1) || (x_type == 1 && terms != 1))
    return hipErrorInvalidValue;
  SeqArgs g{};
  g.d.x1 = x1; g.d.x2 = x2; g.d.w = (const uint8_t*)w; g.d.b1 = b_ih; g.d.b2 = b_hh;
  g.d.M = N; g.d.I1 = I1; g.d.I2 = I2; g.d.H = H; g.d.S = lstm ? 2 * H : H;
  g.d.k1 = I1 / 32; g.d.k2 = (I1 + I2) / 32; g.d.kn = g.d.k2 + H / 32;
  g.h0 = h0; g.done = done; g.seq = h_seq; g.T = T; g.n_cg = H / 8;
  g.ticket = words; g.mark = words + 1; g.limit = limit;
  const long long rows = (long long)T * N, pieces = rows * (H / 4);
  core_seq_fill_kernel<<<(unsigned)(pieces < 256 * 1024 ? (pieces + 255) / 256 : 1024), 256, 0, st>>>(h_seq, rows, H, g.d.S, words, 1 + 2 * N);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (terms == 3) return lstm ? launch_kind<LSTM, X_F32, 3>(g, cus, st) : launch_kind<GRU, X_F32, 3>(g, cus, st);
  if (x_type == 1) return lstm ? launch_kind<LSTM, X_BF16, 1>(g, cus, st) : launch_kind<GRU, X_BF16, 1>(g, cus, st);
  return lstm ? launch_kind<LSTM, X_F32, 1>(g, cus, st) : launch_kind<GRU, X_F32, 1>(g, cus, st);
}

}  // namespace sf
