// Measurement encoder of the full architecture (paper, App. "Model architectures"): device code shared by
// its own launch (k_generic.hip) and the FC layer's (k_dense_split.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sf {

// in [B][n0]; w1 [n0][n1], w2 [n1][n2] (transposed weights); n2 == 0: a single layer; out [B][n2 ? n2 : n1]
struct MeasArgs {
  const float *in, *w1, *b1, *w2, *b2;
  float* out;
  int B, n0, n1, n2;
};

// One or two fully connected + ReLU layers.  A workgroup handles kMeasRows rows; the rows' inputs and
// the hidden activations sit in LDS, every weight is read once per workgroup.  The time is the latency
// of the weight loads, so four groups of threads share the inputs of a layer and the first weights of
// both layers are requested at once; the partial sums meet in LDS.  (One group, eight loads in flight:
// 10 us for 23 -> 128 -> 128 on 333 rows; 5.9 as a launch of its own; beside the FC layer the step is 4.2
// shorter at 333 rows, 5.5 at 16.)
constexpr int kMeasRows = 4;
constexpr int kMeasCols = 128;   // outputs at a time
constexpr int kMeasParts = 4;    // groups of threads along the inputs
constexpr int kMeasThreads = kMeasCols * kMeasParts;

// A thread's first weights of a layer, and its bias: requested for both layers at the kernel's start.
template <int BATCH>
struct MeasFirst {
  float w[BATCH], bias;
  __device__ inline void load(const float* __restrict__ w_t, const float* __restrict__ b, int n_in, int n_out) {
    const int o = min((int)threadIdx.x % kMeasCols, n_out - 1), q = threadIdx.x / kMeasCols;
    const int k0 = n_in * q / kMeasParts, k1 = n_in * (q + 1) / kMeasParts;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) w[u] = w_t[(uint32_t)(max(min(k0 + u, k1 - 1), 0) * n_out + o)];
    bias = b[o];
  }
};

template <int BATCH>
__device__ inline void meas_layer(const float* in, int n_in, const float* __restrict__ w_t, const float* __restrict__ b,
                                  int n_out, MeasFirst<BATCH>& first, float* part, float* hidden, float* out, int rows) {
  const int tid = threadIdx.x, c = tid % kMeasCols, q = tid / kMeasCols;
  const int k0 = n_in * q / kMeasParts, k1 = n_in * (q + 1) / kMeasParts;
  for (int o0 = 0; o0 < n_out; o0 += kMeasCols) {
    const int o = min(o0 + c, n_out - 1);
    if (o0) first.bias = b[o];
    float acc[kMeasRows];
#pragma unroll
    for (int r = 0; r < kMeasRows; ++r) acc[r] = 0.0f;
    for (int i = k0; i < k1; i += BATCH) {
      if (o0 || i != k0)
#pragma unroll
        for (int u = 0; u < BATCH; ++u) first.w[u] = w_t[(uint32_t)(min(i + u, k1 - 1) * n_out + o)];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        // past the end: 0 times the last weight again (the input is the one to leave out: it may be infinite)
#pragma unroll
        for (int r = 0; r < kMeasRows; ++r) {
          const float x = in[r * n_in + i + u];  // (read in any case, see meas_lds: no branches)
          acc[r] = fmaf(i + u < k1 ? x : 0.0f, first.w[u], acc[r]);
        }
        // (no more LDS reads in flight than this: the FC layer's launch has 128 registers in one of its tiles)
        if (u % 8 == 7) __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int r = 0; r < kMeasRows; ++r) part[(q * kMeasRows + r) * kMeasCols + c] = acc[r];
    __syncthreads();
    const int r = q;  // (as many groups as rows)
    float v = first.bias;
#pragma unroll
    for (int p = 0; p < kMeasParts; ++p) v += part[(p * kMeasRows + r) * kMeasCols + c];
    v = fmaxf(v, 0.0f);
    if (o0 + c < n_out) {
      if (hidden)
        hidden[r * n_out + o] = v;
      else if (r < rows)
        out[(size_t)r * n_out + o] = v;
    }
    __syncthreads();
  }
}

// floats of LDS for the rows of a workgroup (a last row is read up to a batch past its end)
constexpr int meas_lds(int n0, int n1) { return kMeasParts * kMeasRows * kMeasCols + kMeasRows * (n0 + n1) + 32; }

// Rows kMeasRows * block .. of it, by kMeasThreads threads.
__device__ inline void meas_rows(const MeasArgs& g, int block, float* lds) {
  static_assert(kMeasParts == kMeasRows, "a group finishes a row");
  float* part = lds;
  float* s_in = lds + kMeasParts * kMeasRows * kMeasCols;  // [kMeasRows][n0]
  float* s_h = s_in + kMeasRows * g.n0;                    // [kMeasRows][n1]
  const int r0 = block * kMeasRows, rows = min(g.B - r0, kMeasRows);
  MeasFirst<8> first1;
  MeasFirst<32> first2;
  first1.load(g.w1, g.b1, g.n0, g.n1);
  if (g.n2 > 0) first2.load(g.w2, g.b2, g.n1, g.n2);
  for (int i = threadIdx.x; i < kMeasRows * g.n0; i += kMeasThreads)
    s_in[i] = i < rows * g.n0 ? g.in[(size_t)r0 * g.n0 + i] : 0.0f;
  __syncthreads();
  meas_layer(s_in, g.n0, g.w1, g.b1, g.n1, first1, part, g.n2 > 0 ? s_h : nullptr, g.out + (size_t)r0 * g.n1, rows);
  if (g.n2 > 0) meas_layer(s_h, g.n1, g.w2, g.b2, g.n2, first2, part, nullptr, g.out + (size_t)r0 * g.n2, rows);
}

}  // namespace sf
