// Recurrent core of the bf16 configurations on the 16-bit MFMA (paper, App. "Model
// architectures": LSTM core of the benchmark model, GRU cells in the large-scale runs).
//
// Same cell arithmetic, reset rule and state layout as the fp32 kernel.  The weights of a
// bf16 configuration are bf16 numbers, the core's input is a bf16 activation (rounded to
// nearest even while it is staged, or handed over as bf16 by the FC kernel, which rounds the
// same way), and the fp32 state h enters the contraction as the
// exact sum of two bf16 numbers, h = hi + lo with hi = bf16(h), lo = bf16(h - hi)
// (relative error below 2^-16): K runs over the input features and then, per 64-wide block
// of h, over its hi part and its lo part, both against the same rows of W_hh (which, like
// the block of h, are fetched once and reused from registers).  The state itself, the gates
// and the blend stay fp32.
//
// v_mfma_f32_32x32x16_bf16: lane l supplies A[i = l%32][k = 8*(l/32) + e] and
// B[k = 8*(l/32) + e][j = l%32].  The weights take the A role (i = hidden unit), the batch
// rows the B role, so a lane ends up with 4 consecutive hidden units of one batch row per
// register quad and the epilogue moves 16-byte pieces of the state.
// Workgroup: 128 batch rows (one 32-row block per wave) x 32 hidden units x all gates:
// four accumulator tiles per wave (GRU r, z, n_x, n_h; LSTM i, f, g, o).  K in chunks of 64
// through double-buffered LDS (pitch 144 bytes), global loads one chunk ahead.
#include <string.h>

#include <mutex>
#include <type_traits>

#include "sf_internal.h"

namespace sf {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;       // K elements per chunk
constexpr int kPitch = 144;   // LDS row pitch in bytes (128 + 16)
constexpr int kBR = 128;      // batch rows per workgroup
constexpr int kBJ = 32;       // hidden units per workgroup

// The gate functions on the hardware's exp2 and reciprocal (about 1 ulp each; no range
// reduction, no division sequence, no branches: sixteen state elements per thread pass through
// here, and with the library routines the epilogue held 40 % of the kernel's instructions).
// exp2 overflows to +inf and underflows to 0, which the reciprocal maps to 0 and 1: the
// limits come out exact.  tanh as (1 - e) / (1 + e) with e = exp(-2|a|) <= 1, sign restored.
__device__ inline float exp_hw(float a) { return __builtin_amdgcn_exp2f(a * 1.44269504088896341f); }
__device__ inline float sigmoid_acc(float a) { return __builtin_amdgcn_rcpf(1.0f + exp_hw(-a)); }
__device__ inline float tanh_acc(float a) {
  const float e = exp_hw(-2.0f * fabsf(a));
  return copysignf((1.0f - e) * __builtin_amdgcn_rcpf(1.0f + e), a);
}

struct RnnBf16Args {
  const void* x1;         // [B][I1], fp32 or (rnn_ring_kernel, I2 == 0) bf16
  const float* x2;        // [B][I2] or null
  const float* h_in;      // state rows of S floats, row index = batch row or ids[row]
  const uint8_t* done;    // [B]
  const uint16_t* w_ih;   // bf16 [G*H][I1 + I2]
  const uint16_t* w_hh;   // bf16 [G*H][H]
  const float* b_ih;      // [G*H]
  const float* b_hh;      // [G*H]
  float* h_out;           // [B][S]
  int B, I1, I2, H;
  const int32_t* ids;
  int n_env;
};

// 8 consecutive fp32 -> 8 bf16, round to nearest even through the packed hardware conversion:
// the values themselves (hi), and with SPLIT also what is left of them, lo = bf16(v - hi)
template <bool SPLIT>
__device__ inline void to_bf16x8(const f32x4& a, const f32x4& b, u32x4& hi_out, u32x4& lo_out) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const f32x2_t p = {v[2 * e], v[2 * e + 1]};
    const unsigned hi = __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf16x2_t));
    hi_out[e] = hi;
    if (SPLIT) {
      const f32x2_t r = {v[2 * e] - __uint_as_float(hi << 16), v[2 * e + 1] - __uint_as_float(hi & 0xFFFF0000u)};
      lo_out[e] = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2_t));
    }
  }
}

// Gates and new state of one batch row m: register 4 q4 + u of a tile holds hidden unit j_lane + 8 q4 + u.  hm: its
// row of the state, reset: that counts as zeros.  (All requests ahead of the first use: one trip to memory, not
// four.)
template <bool LSTM>
__device__ __attribute__((always_inline)) inline void cell_epilogue(const RnnBf16Args& g, const f32x16 (&acc)[4], int m, int hm, bool reset, int j_lane) {
  constexpr int NG = LSTM ? 4 : 3;
  const int H = g.H, S = LSTM ? 2 * H : H;
  f32x4 bi[4][NG], bh[4][NG], prev[4];
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const int j = j_lane + 8 * q4;
    prev[q4] = *(const f32x4*)(g.h_in + (size_t)hm * S + (LSTM ? H : 0) + j);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      bi[q4][q] = *(const f32x4*)(g.b_ih + q * H + j);
      bh[q4][q] = *(const f32x4*)(g.b_hh + q * H + j);
    }
  }
  if (m >= g.B) return;
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const int j = j_lane + 8 * q4;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f}, before = reset ? zero : prev[q4];
    f32x4 hn, cn;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int v = 4 * q4 + u;
      if (LSTM) {
        const float ig = sigmoid_acc(acc[0][v] + bi[q4][0][u] + bh[q4][0][u]);
        const float fg = sigmoid_acc(acc[1][v] + bi[q4][1][u] + bh[q4][1][u]);
        const float gg = tanh_acc(acc[2][v] + bi[q4][2][u] + bh[q4][2][u]);
        const float og = sigmoid_acc(acc[3][v] + bi[q4][NG - 1][u] + bh[q4][NG - 1][u]);
        cn[u] = fg * before[u] + ig * gg;
        hn[u] = og * tanh_acc(cn[u]);
      } else {
        const float r = sigmoid_acc(acc[0][v] + bi[q4][0][u] + bh[q4][0][u]);
        const float z = sigmoid_acc(acc[1][v] + bi[q4][1][u] + bh[q4][1][u]);
        const float n = tanh_acc(acc[2][v] + bi[q4][2][u] + r * (acc[3][v] + bh[q4][2][u]));
        hn[u] = (1.0f - z) * n + z * before[u];
      }
    }
    if (LSTM) *(f32x4*)(g.h_out + (size_t)m * S + H + j) = cn;
    *(f32x4*)(g.h_out + (size_t)m * S + j) = hn;
  }
}

template <bool LSTM>
__global__ __launch_bounds__(256) void rnn_bf16_kernel(RnnBf16Args g) {
  constexpr int NG = LSTM ? 4 : 3;
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * (kBR + NG * kBJ) * kPitch];
  unsigned char* Rs = smem;                       // [2][128][pitch] batch rows
  unsigned char* Ws = smem + 2 * kBR * kPitch;    // [2][NG*32][pitch] weight rows

  const int B = g.B, H = g.H, I = g.I1 + g.I2;
  const int S = LSTM ? 2 * H : H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 31, lh = lane >> 5;
  const int m0 = blockIdx.x * kBR, j0 = blockIdx.y * kBJ;
  const int lrow = tid >> 3, lk8 = (tid & 7) * 8;  // 8 threads x 8 elements per tile row

  int am[4], ah[4];
  bool areset[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int m = m0 + lrow + 32 * r;
    am[r] = m < B ? m : B - 1;  // rows past the end re-read the last row; never stored
    areset[r] = g.done[am[r]] != 0;
    ah[r] = am[r];
    if (g.ids) {
      const int e = g.ids[am[r]];
      const bool ok = (unsigned)e < (unsigned)g.n_env;
      ah[r] = ok ? e : 0;
      areset[r] = areset[r] || !ok;
    }
  }
  const int n1c = g.I1 / kBK, nxc = I / kBK, nhc = H / kBK;

  f32x4 ra[4][2];
  u32x4 rw[NG];
  // K runs over the x chunks and then, per 64-wide block of h, over its hi part and its lo
  // part: the lo chunk reuses the state values and the weight rows that the hi chunk loaded
  // (they stay in registers), so every block of h and of W_hh is fetched once.
  auto gload_x = [&](int c) {
    const int kk = c * kBK + lk8;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* src = c < n1c ? (const float*)g.x1 + (size_t)am[r] * g.I1 + kk
                                 : g.x2 + (size_t)am[r] * g.I2 + (kk - g.I1);
      ra[r][0] = *(const f32x4*)src;
      ra[r][1] = *(const f32x4*)(src + 4);
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
      rw[q] = *(const u32x4*)(g.w_ih + (size_t)(q * H + j0 + lrow) * I + kk);
  };
  auto gload_h = [&](int kb) {
    const int kk = kb * kBK + lk8;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* src = g.h_in + (size_t)ah[r] * S + kk;
      ra[r][0] = *(const f32x4*)src;
      ra[r][1] = *(const f32x4*)(src + 4);
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
      rw[q] = *(const u32x4*)(g.w_hh + (size_t)(q * H + j0 + lrow) * H + kk);
  };
  // rphase: 0 = x values, 1 = hi parts of h, 2 = lo parts of h.  A block of h is split once,
  // when its hi part is stored: the lo words then take the place of the fp32 values in the
  // registers and phase 2 only stores them.
  auto sstore = [&](int buf, int rphase) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      // the reset is applied here, not behind the load (a select there waits for the load)
      const u32x4 zero = {0u, 0u, 0u, 0u};
      u32x4 v, lo;
      if (rphase == 0) {
        to_bf16x8<false>(ra[r][0], ra[r][1], v, lo);
      } else if (rphase == 1) {
        to_bf16x8<true>(ra[r][0], ra[r][1], v, lo);
        ra[r][0] = __builtin_bit_cast(f32x4, lo);
      } else {
        v = __builtin_bit_cast(u32x4, ra[r][0]);
      }
      *(u32x4*)(Rs + (buf * kBR + lrow + 32 * r) * kPitch + lk8 * 2) = (rphase != 0 && areset[r]) ? zero : v;
    }
#pragma unroll
    for (int q = 0; q < NG; ++q)
      *(u32x4*)(Ws + (buf * NG * kBJ + q * kBJ + lrow) * kPitch + lk8 * 2) = rw[q];
  };

  f32x16 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;

  auto compute = [&](int buf, auto xph) {
    const unsigned char* rb = Rs + (buf * kBR + wave * 32 + li) * kPitch + lh * 16;
    const unsigned char* wb = Ws + (buf * NG * kBJ + li) * kPitch + lh * 16;
    constexpr bool xphase = decltype(xph)::value;
#pragma unroll
    for (int ks = 0; ks < kBK / 16; ++ks) {
      const bf16x8 bfrag = __builtin_bit_cast(bf16x8, *(const u32x4*)(rb + ks * 32));
      bf16x8 afrag[NG];
#pragma unroll
      for (int q = 0; q < NG; ++q)
        afrag[q] = __builtin_bit_cast(bf16x8, *(const u32x4*)(wb + q * kBJ * kPitch + ks * 32));
      if (LSTM) {
#pragma unroll
        for (int q = 0; q < NG; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[q], bfrag, acc[q], 0, 0, 0);
      } else {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[0], bfrag, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[1], bfrag, acc[1], 0, 0, 0);
        if (xphase)
          acc[2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[2], bfrag, acc[2], 0, 0, 0);
        else
          acc[3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[2], bfrag, acc[3], 0, 0, 0);
      }
    }
  };

  // Single register set: loads of the next chunk, MFMAs of this one, conversion and LDS
  // store of the next, barrier; `cb` counts chunks (LDS buffer = parity).  One plain loop
  // per accumulator set, no conditions around the loads.
  using Xp = std::true_type;
  using Hp = std::false_type;
  int cb = 0;
  gload_x(0);
  sstore(0, 0);
  __syncthreads();
  for (int c = 0; c + 1 < nxc; ++c, ++cb) {
    gload_x(c + 1);
    compute(cb & 1, Xp{});
    sstore((cb + 1) & 1, 0);
    __syncthreads();
  }
  gload_h(0);  // the last x chunk runs while block 0 of h arrives
  compute(cb & 1, Xp{});
  sstore((cb + 1) & 1, 1);
  __syncthreads();
  ++cb;
  for (int kb = 0; kb + 1 < nhc; ++kb) {
    compute(cb & 1, Hp{});      // hi part of block kb
    sstore((cb + 1) & 1, 2);    // its lo part, from the same registers
    __syncthreads();
    ++cb;
    gload_h(kb + 1);
    compute(cb & 1, Hp{});      // lo part of block kb
    sstore((cb + 1) & 1, 1);    // hi part of block kb + 1
    __syncthreads();
    ++cb;
  }
  compute(cb & 1, Hp{});
  sstore((cb + 1) & 1, 2);
  __syncthreads();
  ++cb;
  compute(cb & 1, Hp{});

  const int m = m0 + wave * 32 + li;
  int hm = min(m, B - 1);
  bool reset = g.done[hm] != 0;
  if (g.ids) {
    const int e = g.ids[hm];
    const bool ok = (unsigned)e < (unsigned)g.n_env;
    hm = ok ? e : 0;
    reset = reset || !ok;
  }
  cell_epilogue<LSTM>(g, acc, m, hm, reset, j0 + 4 * lh);
}

// The same with features in bf16, out of a ring in LDS (see k_fc16.hip).  The kernel above has one chunk on its
// way and two barriers' worth of conversions per chunk: 3.2 k cycles per chunk and CU at 768 of products.  Taking
// these rows, too, it made steps of a network of 512 features and units 59.6 us at 700 rows (52.9 with this one), 65.5 at 1024
// (58.8), 80.8 at 1500 (77.3), 92.6 at 2048 (89.6), 143.8 at 4096 (141.3; the launch 34.6 -> 31.2), 274 at
// 8192 (269).  What bounds it now: with few rows the way from L2 into LDS (7 to 10 TB/s).  In the tile of most rows (128 x 64:
// beyond 2048 rows of 512 units, 6.5 TB/s) the ring is four chunks deep, since a slot has room for a chunk of the fp32
// state, of which features fill half: two chunks are on their way, and each barrier waits for both.  k_fc16.hip draws 12
// TB/s over the same path, so that this is exposed latency.  Here
// chunks of 32 numbers of K go straight to LDS, two per barrier, kDepth - 2 ahead (kDepth 8, 8, 4 in the tiles of 64 x 32, 64 x 64,
// 128 x 64; LSTM 8, 6, 4): bf16 features, then the fp32 state, which is
// split into its two bf16 numbers by the wave that reads it (twice: two tiles of units) and zeroed there where
// an episode begins; each with the weights of its columns.  RT x UT waves of 32 rows x 32 units x all gates.
// Rows of features and weights are 64 bytes (four pieces, exchanged by r / 4), of the state 128 (eight, by
// r / 2): 16 neighbouring rows read different banks.
typedef __attribute__((address_space(3))) unsigned char LdsByte;
constexpr int kRingLds = 160 * 1024;

__device__ __attribute__((always_inline)) inline void load_lds(__amdgpu_buffer_rsrc_t from, LdsByte* to, int at, int k) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, to, 16, at, k, 0, 0);
}
__device__ __attribute__((always_inline)) inline void load_lds(const uint8_t* from, LdsByte* to) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from, to, 16, 0, 0);
}

template <bool LSTM, int RT, int UT>
struct Ring {
  static constexpr int NG = LSTM ? 4 : 3, NW = RT * UT;
  static constexpr int A = RT * 32 * 128;             // bytes of a chunk's rows (features: the first half)
  static constexpr int CH = A + NG * UT * 32 * 64;
  static constexpr int kDepth = kRingLds / CH < 8 ? kRingLds / CH / 2 * 2 : 8;
  static constexpr int AX = 2 * RT / NW;              // load instructions of a wave: features, state (twice as many),
  static constexpr int WI = NG * UT * 2;              // and weights, of all waves
  static constexpr int WL = (WI + NW - 1) / NW;
  static_assert(AX * NW == 2 * RT, "whole instructions");
  static_assert(kDepth >= 4 && (2 * AX + WL) * (kDepth - 4) < 64, "as many as the counter holds");
};

template <bool LSTM, int RT, int UT>
__global__ __launch_bounds__(64 * RT * UT, 2) void rnn_ring_kernel(RnnBf16Args g) {
  using R = Ring<LSTM, RT, UT>;
  constexpr int NG = R::NG, NW = R::NW, kDepth = R::kDepth, CH = R::CH, AX = R::AX, WL = R::WL;
  extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
  LdsByte* const base = (LdsByte*)ring;
  const int B = g.B, H = g.H, S = LSTM ? 2 * H : H;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const int rt = wave / UT, ut = wave % UT;

  // tiles in runs of neighbours per XCD: the units of a row tile read the same rows out of its L2
  const int n_ut = H / (32 * UT), n_tiles = (B + 32 * RT - 1) / (32 * RT) * n_ut, per_xcd = (n_tiles + 7) / 8;
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= n_tiles) return;
  const int m0 = tile / n_ut * (32 * RT), j0 = tile % n_ut * (32 * UT);

  // the state's row of batch row m, and whether it enters as zeros
  auto state_row = [&](int m, bool& zero) {
    zero = g.done[m] != 0;
    if (!g.ids) return m;
    const int e = g.ids[m];
    const bool ok = (unsigned)e < (unsigned)g.n_env;
    zero = zero || !ok;
    return ok ? e : 0;
  };
  bool reset;
  const int hm = state_row(min(m0 + 32 * rt + li, B - 1), reset);
  const unsigned keep = reset ? 0u : ~0u;

  // ---- what this wave asks for: instruction i of a chunk is 16 rows (state: 8) of 64 lanes' pieces ----
  const int last = min(B - m0, 32 * RT) - 1;  // (past the last row: that row again, never stored)
  const int x_pitch = 2 * g.I1, h_pitch = 2 * H;
  const auto xs = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint8_t*)g.x1 + (size_t)m0 * x_pitch), 0, (last + 1) * x_pitch, 0x00027000);
  const auto wis = __builtin_amdgcn_make_buffer_rsrc((void*)g.w_ih, 0, NG * H * x_pitch, 0x00027000);
  const auto whs = __builtin_amdgcn_make_buffer_rsrc((void*)g.w_hh, 0, NG * H * h_pitch, 0x00027000);
  int x_at[AX], wi_at[WL], wh_at[WL];
  const uint8_t* h_at[2 * AX];
#pragma unroll
  for (int j = 0; j < AX; ++j) {
    const int r = 16 * (wave + NW * j) + (lane >> 2);
    x_at[j] = min(r, last) * x_pitch + (((lane & 3) ^ ((r >> 2) & 3)) << 4);
  }
#pragma unroll
  for (int j = 0; j < 2 * AX; ++j) {
    const int r = 8 * (wave + NW * j) + (lane >> 3);
    bool unused;
    const int row = state_row(m0 + min(r, last), unused);
    h_at[j] = (const uint8_t*)(g.h_in + (size_t)row * S) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int j = 0; j < WL; ++j) {
    const int r = 16 * min(wave + NW * j, R::WI - 1) + (lane >> 2);  // row of the chunk: gate, unit
    const int row = r / (32 * UT) * H + j0 + r % (32 * UT), piece = ((lane & 3) ^ ((r >> 2) & 3)) << 4;
    wi_at[j] = row * x_pitch + piece;
    wh_at[j] = row * h_pitch + piece;
  }
  const int nx = g.I1 / 32, n = nx + H / 32;
  const bool spare = R::WI % NW != 0 && wave >= R::WI % NW;  // one weight instruction fewer
  auto request = [&](int c, int slot) __attribute__((always_inline)) {
    LdsByte* const to = base + (slot * CH + 1024 * wave);
    c = min(c, n - 1);  // (past the end: the last one again, for no use)
    if (c < nx) {
#pragma unroll
      for (int j = 0; j < AX; ++j) load_lds(xs, to + 1024 * NW * j, x_at[j], 64 * c);
#pragma unroll
      for (int j = 0; j < WL; ++j)
        if (j + 1 < WL || !spare) load_lds(wis, to + R::A + 1024 * NW * j, wi_at[j], 64 * c);
    } else {
      c -= nx;
#pragma unroll
      for (int j = 0; j < 2 * AX; ++j) load_lds(h_at[j] + 128 * c, to + 1024 * NW * j);
#pragma unroll
      for (int j = 0; j < WL; ++j)
        if (j + 1 < WL || !spare) load_lds(whs, to + R::A + 1024 * NW * j, wh_at[j], 64 * c);
    }
  };
#pragma unroll
  for (int c = 0; c < kDepth - 2; ++c) request(c, c);

  // ---- operands: piece 2 s + lh of features and weights, pieces 4 s + 2 lh, + 1 of the state ----
  const unsigned lds0 = (unsigned)(size_t)base;
  unsigned f64[2], f128[2][2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    f64[s] = lds0 + li * 64 + (((2 * s + lh) ^ ((li >> 2) & 3)) << 4);
#pragma unroll
    for (int p = 0; p < 2; ++p) f128[s][p] = lds0 + 32 * rt * 128 + li * 128 + (((4 * s + 2 * lh + p) ^ ((li >> 1) & 7)) << 4);
  }
  const unsigned x_from = 32 * rt * 64, w_from = R::A + 32 * ut * 64;
  constexpr int kGate = 32 * UT * 64;  // bytes between the gates' rows

  f32x16 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
  auto mfma = [&](const u32x4& w, const u32x4& x, f32x16& c) __attribute__((always_inline)) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
  };
  // reads and their wait in one block (the compiler would wait for every load to LDS ahead of a read): the
  // gates' weights of both halves of a chunk, and NV other pieces
  auto read = [&](unsigned w0, unsigned w1, const unsigned (&from)[4], auto nv, u32x4 (&w)[2][4], u32x4 (&v)[4]) __attribute__((always_inline)) {
    constexpr int NV = decltype(nv)::value;
    if constexpr (LSTM && NV == 4)
      asm volatile(
          "ds_read_b128 %0, %12\n\t"
          "ds_read_b128 %1, %12 offset:%c18\n\t"
          "ds_read_b128 %2, %12 offset:%c19\n\t"
          "ds_read_b128 %3, %12 offset:%c20\n\t"
          "ds_read_b128 %8, %14\n\t"
          "ds_read_b128 %9, %15\n\t"
          "ds_read_b128 %4, %13\n\t"
          "ds_read_b128 %5, %13 offset:%c18\n\t"
          "ds_read_b128 %6, %13 offset:%c19\n\t"
          "ds_read_b128 %7, %13 offset:%c20\n\t"
          "ds_read_b128 %10, %16\n\t"
          "ds_read_b128 %11, %17\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[0][3]), "=&v"(w[1][0]), "=&v"(w[1][1]),
            "=&v"(w[1][2]), "=&v"(w[1][3]), "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
          : "v"(w0), "v"(w1), "v"(from[0]), "v"(from[1]), "v"(from[2]), "v"(from[3]), "i"(kGate), "i"(2 * kGate), "i"(3 * kGate)
          : "memory");
    else if constexpr (LSTM)
      asm volatile(
          "ds_read_b128 %0, %10\n\t"
          "ds_read_b128 %1, %10 offset:%c14\n\t"
          "ds_read_b128 %2, %10 offset:%c15\n\t"
          "ds_read_b128 %3, %10 offset:%c16\n\t"
          "ds_read_b128 %8, %12\n\t"
          "ds_read_b128 %4, %11\n\t"
          "ds_read_b128 %5, %11 offset:%c14\n\t"
          "ds_read_b128 %6, %11 offset:%c15\n\t"
          "ds_read_b128 %7, %11 offset:%c16\n\t"
          "ds_read_b128 %9, %13\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[0][3]), "=&v"(w[1][0]), "=&v"(w[1][1]),
            "=&v"(w[1][2]), "=&v"(w[1][3]), "=&v"(v[0]), "=&v"(v[1])
          : "v"(w0), "v"(w1), "v"(from[0]), "v"(from[1]), "i"(kGate), "i"(2 * kGate), "i"(3 * kGate)
          : "memory");
    else if constexpr (NV == 4)
      asm volatile(
          "ds_read_b128 %0, %10\n\t"
          "ds_read_b128 %1, %10 offset:%c16\n\t"
          "ds_read_b128 %2, %10 offset:%c17\n\t"
          "ds_read_b128 %6, %12\n\t"
          "ds_read_b128 %7, %13\n\t"
          "ds_read_b128 %3, %11\n\t"
          "ds_read_b128 %4, %11 offset:%c16\n\t"
          "ds_read_b128 %5, %11 offset:%c17\n\t"
          "ds_read_b128 %8, %14\n\t"
          "ds_read_b128 %9, %15\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[1][0]), "=&v"(w[1][1]), "=&v"(w[1][2]),
            "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
          : "v"(w0), "v"(w1), "v"(from[0]), "v"(from[1]), "v"(from[2]), "v"(from[3]), "i"(kGate), "i"(2 * kGate)
          : "memory");
    else
      asm volatile(
          "ds_read_b128 %0, %8\n\t"
          "ds_read_b128 %1, %8 offset:%c12\n\t"
          "ds_read_b128 %2, %8 offset:%c13\n\t"
          "ds_read_b128 %6, %10\n\t"
          "ds_read_b128 %3, %9\n\t"
          "ds_read_b128 %4, %9 offset:%c12\n\t"
          "ds_read_b128 %5, %9 offset:%c13\n\t"
          "ds_read_b128 %7, %11\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(w[0][0]), "=&v"(w[0][1]), "=&v"(w[0][2]), "=&v"(w[1][0]), "=&v"(w[1][1]), "=&v"(w[1][2]),
            "=&v"(v[0]), "=&v"(v[1])
          : "v"(w0), "v"(w1), "v"(from[0]), "v"(from[1]), "i"(kGate), "i"(2 * kGate)
          : "memory");
  };
  auto wait = [&](auto v) __attribute__((always_inline)) {
    constexpr int V = decltype(v)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70 | (V & 15) | (V >> 4) << 14);
  };
  // Two chunks have come once at most the instructions of the kDepth - 4 chunks behind them are on their way
  // (features: counted as if all of those were features, too; ones of the state have more instructions).
  auto arrived = [&](auto per_a) __attribute__((always_inline)) {
    constexpr int P = decltype(per_a)::value;
    if (spare)
      wait(std::integral_constant<int, (P + WL - 1) * (kDepth - 4)>{});
    else
      wait(std::integral_constant<int, (P + WL) * (kDepth - 4)>{});
    __builtin_amdgcn_s_barrier();  // ... everywhere; the two before them have been read
    __builtin_amdgcn_sched_barrier(0);
  };

  int slot = 0;
  auto advance = [&](int c) __attribute__((always_inline)) {
    const int before = slot == 0 ? kDepth - 2 : slot - 2;
    request(c + kDepth - 2, before);
    request(c + kDepth - 1, before + 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto next = [&]() { slot = slot + 2 == kDepth ? 0 : slot + 2; };
  int c = 0;
  for (; c < nx; c += 2) {
    arrived(std::integral_constant<int, AX>{});
    advance(c);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const unsigned at = (slot + half) * CH, from[4] = {f64[0] + at + x_from, f64[1] + at + x_from};
      u32x4 w[2][4], x[4];
      read(f64[0] + at + w_from, f64[1] + at + w_from, from, std::integral_constant<int, 2>{}, w, x);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < NG; ++q) mfma(w[s][q], x[s], acc[q]);
    }
    next();
  }
  // (the order of the kernel above: of 64 numbers first the hi parts, then the lo parts, with the weights kept)
  for (; c < n; c += 2) {
    arrived(std::integral_constant<int, 2 * AX>{});
    advance(c);
    u32x4 w[2][2][4], lo[2][2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const unsigned at = (slot + half) * CH;
      const unsigned from[4] = {f128[0][0] + at, f128[0][1] + at, f128[1][0] + at, f128[1][1] + at};
      u32x4 v[4];
      read(f64[0] + at + w_from, f64[1] + at + w_from, from, std::integral_constant<int, 4>{}, w[half], v);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        u32x4 hi;
        to_bf16x8<true>(__builtin_bit_cast(f32x4, v[2 * s] & keep), __builtin_bit_cast(f32x4, v[2 * s + 1] & keep), hi, lo[half][s]);
#pragma unroll
        for (int q = 0; q < NG; ++q) mfma(w[half][s][q], hi, acc[!LSTM && q == 2 ? 3 : q]);
      }
    }
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int q = 0; q < NG; ++q) mfma(w[half][s][q], lo[half][s], acc[!LSTM && q == 2 ? 3 : q]);
    next();
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // (nothing writes to LDS behind this workgroup's end)
  cell_epilogue<LSTM>(g, acc, m0 + 32 * rt + li, hm, reset, j0 + 32 * ut + 4 * lh);
}

template <bool LSTM, int RT, int UT>
hipError_t launch_ring_t(const RnnBf16Args& g, hipStream_t st) {
  auto kern = rnn_ring_kernel<LSTM, RT, UT>;
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&] {
    attr_status = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kRingLds);
  });
  if (attr_status != hipSuccess) return attr_status;
  using R = Ring<LSTM, RT, UT>;
  const int n_tiles = (g.B + 32 * RT - 1) / (32 * RT) * (g.H / (32 * UT));
  kern<<<(unsigned)((n_tiles + 7) / 8 * 8), 64 * R::NW, R::kDepth * R::CH, st>>>(g);
  return hipGetLastError();
}
template <bool LSTM>
hipError_t launch_ring(const RnnBf16Args& g, hipStream_t st) {
  // the smallest tile whose grid is one round of workgroups
  if ((g.B + 63) / 64 * (g.H / 32) <= 256) return launch_ring_t<LSTM, 2, 1>(g, st);
  if ((g.B + 63) / 64 * (g.H / 64) <= 256) return launch_ring_t<LSTM, 2, 2>(g, st);
  return launch_ring_t<LSTM, 4, 2>(g, st);
}

}  // namespace

// Every piece of the input and the state width must be whole 64-wide K chunks.
bool rnn_bf16_supported(int I1, int I2, int H) {
  return I1 > 0 && (I1 % kBK) == 0 && (I2 % kBK) == 0 && (H % kBK) == 0;
}

// bf16 bits of weights that are bf16 numbers already (rounded to nearest even otherwise)
void rnn_bf16_pack(const float* w, size_t n, std::vector<uint16_t>& out) {
  out.resize(n);
  for (size_t i = 0; i < n; ++i) {
    uint32_t u;
    memcpy(&u, &w[i], 4);
    out[i] = (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
  }
}

// x1_bf16: x1 holds bf16 values (only without a second input)
hipError_t launch_rnn_bf16(int lstm, int B, int I1, int I2, int H, const void* x1, int x1_bf16,
                           const float* x2, const float* h_in, const uint8_t* done,
                           const uint16_t* w_ih, const uint16_t* w_hh, const float* b_ih,
                           const float* b_hh, float* h_out, const int32_t* ids, int n_env,
                           hipStream_t st) {
  if (B == 0) return hipSuccess;
  if (x1_bf16 && x2) return hipErrorInvalidValue;
  RnnBf16Args g;
  g.x1 = x1; g.x2 = x2; g.h_in = h_in; g.done = done;
  g.w_ih = w_ih; g.w_hh = w_hh; g.b_ih = b_ih; g.b_hh = b_hh; g.h_out = h_out;
  g.B = B; g.I1 = I1; g.I2 = x2 ? I2 : 0; g.H = H; g.ids = ids; g.n_env = n_env;
  if (x1_bf16) return lstm ? launch_ring<true>(g, st) : launch_ring<false>(g, st);
  dim3 grid((B + kBR - 1) / kBR, H / kBJ);
  if (lstm)
    rnn_bf16_kernel<true><<<grid, 256, 0, st>>>(g);
  else
    rnn_bf16_kernel<false><<<grid, 256, 0, st>>>(g);
  return hipGetLastError();
}

}  // namespace sf
