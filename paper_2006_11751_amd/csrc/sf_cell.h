// Gate functions of the recurrent cells and the layout of their packed weights (device code, shared by
// k_dense_split.hip and k_core_seq.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "sf_exchange.h"
#include "sf_meas.h"

namespace sf {

enum Kind { FC = 0, GRU = 1, LSTM = 2 };
enum XType { X_F32 = 0, X_BF16 = 1, X_F16 = 2, X_ROUND = 3 };  // X_ROUND: fp32, one bf16 term is used

__device__ inline float sigmoid_acc(float a) { return 1.0f / (1.0f + expf(-a)); }
// (1 - e) / (1 + e) with e = exp(-2|a|), sign restored: e <= 1, nothing overflows
__device__ inline float tanh_acc(float a) {
  const float e = expf(-2.0f * fabsf(a));
  return copysignf((1.0f - e) / (1.0f + e), a);
}

// (The contractions are written out: left to the compiler, a cell's bits would depend on the tile it is
// computed in.)
__device__ inline float gru_gates(const float (&sum)[4], const float (&bias)[2][4], float prev) {
  const float rg = sigmoid_acc(sum[0] + (bias[0][0] + bias[1][0]));
  const float z = sigmoid_acc(sum[1] + (bias[0][1] + bias[1][1]));
  const float n = tanh_acc(fmaf(rg, sum[3] + bias[1][2], sum[2] + bias[0][2]));
  return fmaf(z, prev, (1.0f - z) * n);
}
__device__ inline float lstm_gates(const float (&sum)[4], const float (&bias)[2][4], float prev, float& cell) {
  const float ig = sigmoid_acc(sum[0] + (bias[0][0] + bias[1][0]));
  const float fg = sigmoid_acc(sum[1] + (bias[0][1] + bias[1][1]));
  const float gg = tanh_acc(sum[2] + (bias[0][2] + bias[1][2]));
  const float og = sigmoid_acc(sum[3] + (bias[0][3] + bias[1][3]));
  cell = fmaf(fg, prev, ig * gg);
  return og * tanh_acc(cell);
}
// a state row: [h] (GRU), [h | c] (LSTM); prev: the unit's h or c
__device__ inline void cell_gru(float* o, int unit, const float (&sum)[4], const float (&bias)[2][4], float prev) {
  o[unit] = gru_gates(sum, bias, prev);
}
__device__ inline void cell_lstm(float* o, int H, int unit, const float (&sum)[4], const float (&bias)[2][4], float prev) {
  float cn;
  const float h = lstm_gates(sum, bias, prev, cn);
  o[H + unit] = cn;
  o[unit] = h;
}

// Bytes of one K step and term of a column group: FC 16 columns; cells 8 units, the gates in
// columns [r z | n] (the 8 n columns of each lane group alone) or [i f | g o].
constexpr int group_bytes(int kind) { return kind == FC ? 1024 : kind == GRU ? 1536 : 2048; }

__device__ inline bool finite(float v) { return fabsf(v) < INFINITY; }
constexpr bool in_f32(int xt) { return xt == X_F32 || xt == X_ROUND; }

struct DenseArgs {
  const void* x1;       // [M][I1] fp32 or 16-bit
  const float* x2;      // [M][I2] or null (cells)
  const float* h_in;    // state rows of S floats, row index = row or ids[row] (cells)
  const uint8_t* done;  // [M] (cells)
  const int32_t* ids;   // [M] or null
  const uint8_t* w;     // packed weights
  const float* b1;      // FC: [N]; cells: b_ih [G*H]
  const float* b2;      // cells: b_hh [G*H]
  void* out;            // FC: [M][N]; cells: state rows [M][S]
  int M, I1, I2, H, S, n_env;
  int N;                // FC outputs
  int k1, k2, kn;       // K steps (of 32): of x1, of x1 and x2, all
  int n_rt, n_cg;       // workgroups along the rows / the columns
  int xcd_rows;         // the 8 XCDs as 2^xcd_rows x 2^(3 - xcd_rows) blocks of
  int per_rt, per_cg;   // per_rt x per_cg workgroups
  uint32_t rcp_cg;      // 2^32 / per_cg, rounded up
  int blocks;           // FC: workgroups ahead of those of the measurement layers
  MeasArgs meas;        // B = 0: none
};

// The sums of one row that holds an infinity or a NaN, or of a row whose sum came out as one, in plain
// fp32 arithmetic: the products of such a number with the terms of a weight do not add up to its
// product with the weight, and neither do those of terms whose largest product overflows.  q: gate
// (FC: 0), n: unit (FC: output); the n gate of a GRU has its sums over the features (n_x) and the
// state (n_h) apart.  EX: the features are another workgroup's of the same launch (sf_exchange.h).
template <int KIND, int XT, int PB, bool EX = false>
__device__ inline __attribute__((always_inline)) float plain_sum(const DenseArgs& g, int m, int sm, bool reset, int q, int n, int k_from, int k_to) {
  constexpr int GB = group_bytes(KIND);
  constexpr int C = KIND == FC ? 16 : 8;
  float sum = 0.0f;
  for (int k = 32 * k_from; k < 32 * k_to; ++k) {
    const int s = k >> 5, lg = (k >> 3) & 3, e = k & 7;
    float x;
    if (s < g.k1) {
      if (EX && in_f32(XT))
        x = load_float((const float*)g.x1 + (size_t)m * g.I1 + k);
      else if (EX)
        x = __builtin_bit_cast(float, load_word((const unsigned*)g.x1 + ((size_t)m * g.I1 + k) / 2) << (k & 1 ? 0 : 16) & 0xFFFF0000u);
      else if (in_f32(XT))
        x = ((const float*)g.x1)[(size_t)m * g.I1 + k];
      else if (XT == X_BF16)
        x = __builtin_bit_cast(float, (unsigned)((const uint16_t*)g.x1)[(size_t)m * g.I1 + k] << 16);
      else
        x = (float)((const _Float16*)g.x1)[(size_t)m * g.I1 + k];
    } else if (s < g.k2) {
      x = g.x2[(size_t)m * g.I2 + (k - 32 * g.k1)];
    } else {
      x = reset ? 0.0f : g.h_in[(size_t)sm * g.S + (k - 32 * g.k2)];
    }
    if (XT == X_ROUND && s < g.k2) x = (float)(__bf16)x;
    int slot;
    if (KIND == FC)
      slot = lg * 16 + n % C;
    else
      slot = KIND == LSTM || q < 2 ? (q >> 1) * 64 + lg * 16 + (q & 1) * 8 + n % C : 64 + lg * 8 + n % C;
    const uint8_t* at = g.w + ((size_t)(n / C) * g.kn + s) * PB * GB + slot * 16 + e * 2;
    float w;
    if (XT == X_F16) {
      w = (float)*(const _Float16*)at;
    } else {
      w = 0.0f;
      for (int p = PB - 1; p >= 0; --p) w += __builtin_bit_cast(float, (unsigned)*(const uint16_t*)(at + p * GB) << 16);
    }
    sum = fmaf(x, w, sum);
  }
  return sum;
}
template <int KIND, int XT, int PB, bool EX = false>
__device__ inline __attribute__((always_inline)) void plain_sums(const DenseArgs& g, int m, bool reset, int n, float (&sum)[4]) {
  const int sm = g.ids && !reset ? g.ids[m] : m;  // (a reset row's state is not read)
  if (KIND == FC) {
    sum[0] = plain_sum<KIND, XT, PB, EX>(g, m, sm, reset, 0, n, 0, g.kn);
  } else {
    for (int q = 0; q < (KIND == LSTM ? 4 : 2); ++q) sum[q] = plain_sum<KIND, XT, PB, EX>(g, m, sm, reset, q, n, 0, g.kn);
    if (KIND == GRU) {
      sum[2] = plain_sum<KIND, XT, PB, EX>(g, m, sm, reset, 2, n, 0, g.k2);
      sum[3] = plain_sum<KIND, XT, PB, EX>(g, m, sm, reset, 2, n, g.k2, g.kn);
    }
  }
}

}  // namespace sf
