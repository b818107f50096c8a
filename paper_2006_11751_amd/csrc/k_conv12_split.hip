// First and second convolution of the plain encoder in fp32 configurations as one kernel (paper, App.
// "Model architectures": the convolutional encoder), so that the first layer's output (17 x 31 x 32
// values per frame, 68 KB, the largest tensor of the step) never leaves the compute unit.
//
// The arithmetic is that of the two separate kernels: the first layer on the int8 matrix instructions
// against three fixed-point digit planes (k_conv1_i8.hip), its ReLU'd results scaled and written as two
// fp16 terms, the second layer as three products of terms on the 16-bit matrix instructions
// (k_conv_image_split.hip; the small products in an accumulator of their own).  Only the order of the
// second layer's sum differs: filter rows 0, 1 and rows 2, 3 are summed apart and added.
//
// A workgroup of eight waves, one per CU, walks frames b, b + gridDim.x, ...  Per frame:
//   1. the planar byte frame is in LDS (sign-flipped: byte - 128 as int8); the next frame's bytes are
//      requested into registers;
//   2. first layer: tiles of 16 pixels x 16 channels, wave w the channels 16 (w % 2) .. and tiles w / 2,
//      w / 2 + 4, ...; both terms go to a channels-last image in LDS; barrier;
//   3. second layer: wave w the channels 16 (w % 4) .. of all MT tiles of 16 pixels, over half of the
//      filter (K split in two: the banks of both layers then stay in registers, 64 + 36 of them, while
//      all eight waves work on one frame); half of the tiles' sums go to LDS for the wave that has the
//      other half of K; the next frame's bytes go to LDS; barrier;
//   4. the two halves are added; bias, ReLU, one 16-byte store of four channels per lane and tile.
// Tiles of 16 pixels of the flat pixel index fill the matrix instructions (33 tiles of 527 pixels, no
// row remainders), and weights as the A operand leave four neighbouring channels of a pixel in a lane:
// 8-byte LDS writes.
//
// What bounds it: vector-ALU work of the first layer's epilogue (ten instructions per value) and the
// matrix instructions of the second (5.4 k cycles per frame); 4 frames per CU at B = 1024.
//
// v_mfma_i32_16x16x64_i8: lane l supplies 16 bytes of A[i = l%16] and of B[j = l%16], the k block l/16;
// v_mfma_f32_16x16x32_f16: A[i = l%16][k = 8*(l/16) + e], B[k][j = l%16]; both: D[i][j] sits in lane
// j + 16*(i/4), register i%4.
#include <mutex>
#include <type_traits>

#include "sf_internal.h"

namespace sf {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// a frame's address is a multiple of four bytes only; one load instruction all the same
typedef u32x4 u32x4_any __attribute__((aligned(4)));

constexpr int kNT = 512;
constexpr int kCin = 3, kK1 = 8, kS1 = 4, kC1 = 32;  // first layer: planes, filter, stride, channels
constexpr int kK2 = 4, kS2 = 2, kC2 = 64;            // second layer: filter, stride, channels
constexpr int kMaxTiles = 7;                         // 16-pixel tiles of the second layer
constexpr int kP4 = kC1 / 4 + 1;                     // image pixel in 16-byte pieces: both terms and padding
constexpr int kPitch = 160;                          // byte-frame row in LDS, see layout()
constexpr int kNV = 4;                               // 16-byte pieces of a byte frame per thread
constexpr int kG2 = kK2 * kK2 / 2;                   // filter taps of a wave
constexpr size_t kMaxLds = 160 * 1024;
constexpr float kInvRadix2 = 1.0f / 64516.0f;

struct __attribute__((packed, aligned(4))) U2 {
  uint32_t x, y;
};

struct Args {
  const uint8_t* obs;    // [B][3][H][W]
  const int* wpk1;       // digit planes of the first bank, lane order of k_conv1_i8.hip
  const float* scale1;   // [32]
  const float* bias1;    // [32]
  const u32x4* wpk2;     // [4][16][2][64] lane operands of the second bank
  const float* scale2;   // [32] input scales, [64] inverse output scales, 1 if the split is not admitted
  const float* w32;      // [64][4][4][32]
  const float* bias2;    // [64]
  float* mid;            // [B][Ho1*Wo1][32]: for the fallback
  float* out;            // [B][Ho2*Wo2][64]
  int B, H, W, Ho1, Wo1, Ho2, Wo2;
  int row_stride;        // image row in pieces
  int image_at, sums_at, bank_at; // LDS offsets
  int rcp_wo2, rcp_row;  // x / d = x * rcp >> 16 for Wo2, W / 16
  int parts;             // workgroups per frame
  ExchangePrep prep;     // with several workgroups per frame: work for a later launch (sf_exchange.h)
};

int reciprocal(int d) { return (65536 + d - 1) / d; }  // exact for x * d < 65536

// MT: 16-pixel tiles of the second layer per workgroup.  Few frames are dealt to two or four workgroups
// each, by rows of the second layer's output: a workgroup then takes the image rows that these need (the
// first layer's rows at a border are computed twice) and MT = 4 or 2 tiles.
template <int MT>
__global__ __launch_bounds__(kNT, 2) void conv12_split_kernel(Args g) {
  constexpr bool WHOLE = MT == kMaxTiles;
  constexpr int OWN0 = (MT + 1) / 2;  // tiles finished by the first half of the waves
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  uint8_t* const image = lds + g.image_at;
  f32x4* const sums = (f32x4*)(lds + g.sums_at);  // [4][MT][64]

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lp = lane & 15, lg = lane >> 4;
  const int half1 = wave & 1;                  // first layer: channel half
  const int ct = wave & 3, kh = wave >> 2;     // second layer: channel tile, half of the filter

  // rows [row0, row0 + n2) of the second layer's output, n1 of the first layer's, in_rows of the image
  const int part = WHOLE ? 0 : (int)blockIdx.x % g.parts;
  const int row0 = WHOLE ? 0 : part * g.Ho2 / g.parts;
  const int n2 = WHOLE ? g.Ho2 : (part + 1) * g.Ho2 / g.parts - row0;
  const int n1 = WHOLE ? g.Ho1 : kS2 * (n2 - 1) + kK2;
  const int in_rows = WHOLE ? g.H : kS1 * (n1 - 1) + kK1;
  const int first_frame = WHOLE ? (int)blockIdx.x : (int)blockIdx.x / g.parts;
  const int frame_step = WHOLE ? (int)gridDim.x : (int)gridDim.x / g.parts;  // (the same part of every frame)

  const int row_pieces = g.W >> 4, pieces = kCin * in_rows * row_pieces;
  u32x4 fv[kNV];
  auto load_frame = [&](int b) {
    const uint8_t* src = g.obs + (size_t)b * ((size_t)kCin * g.H * g.W);
    int first = tid;
    asm volatile("" : "+v"(first));  // (opaque: the places are computed in place, not kept)
#pragma unroll
    for (int u = 0; u < kNV; ++u) {
      const int f = min(first + kNT * u, pieces - 1);
      uint32_t at = 16u * (uint32_t)f;
      if (!WHOLE) {
        const int plane = (f >= in_rows * row_pieces) + (f >= 2 * in_rows * row_pieces);
        at += (uint32_t)((plane * (g.H - in_rows) + kS1 * kS2 * row0) * g.W);
      }
      fv[u] = *(const u32x4_any*)(src + at);
    }
  };
  auto store_frame = [&]() {
    int first = tid;
    asm volatile("" : "+v"(first));
#pragma unroll
    for (int u = 0; u < kNV; ++u) {
      const int f = min(first + kNT * u, pieces - 1), row = f * g.rcp_row >> 16;
      *(u32x4*)(lds + (row * kPitch + (f - row * row_pieces) * 16)) = fv[u] ^ 0x80808080u;
    }
  };
  load_frame(first_frame);

  // ---- the first bank in LDS: [channel half][channel][digit] operands of 64 lanes ----
  u32x4* const bank1 = (u32x4*)(lds + g.bank_at);
  {
    // (all requests ahead of the first store: one trip to memory)
    constexpr int N = 2 * kCin * 3 * 64, NB = (N + kNT - 1) / kNT;
    u32x4 v[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int i = min(tid + kNT * j, N - 1), l = i & 63, d = (i >> 6) % 3, s = (i >> 6) / 3 % 3, half = (i >> 6) / 9;
      const int* from = g.wpk1 + ((2 * s + (l >> 5)) * 3 + d) * (4 * 64) + 32 * ((l >> 4) & 1) + 16 * half + (l & 15);
      v[j] = u32x4{(unsigned)from[0], (unsigned)from[64], (unsigned)from[128], (unsigned)from[192]};
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
      if (tid + kNT * j < N) bank1[tid + kNT * j] = v[j];
  }
  // its scales and bias, the second layer's input scales (powers of two: the same bits) folded in
  float* const affine1 = (float*)(bank1 + 2 * kCin * 3 * 64);  // [2][32]
  if (tid < 2 * kC1) affine1[tid] = (tid < kC1 ? g.scale1 : g.bias1)[tid % kC1] * g.scale2[tid % kC1];
  // ---- operands that stay in registers ----
  const int c1 = 16 * half1 + 4 * lg, c2 = 16 * ct + 4 * lg;  // this lane's four channels
  u32x4 wf[kG2][2];
#pragma unroll
  for (int t = 0; t < kG2; ++t)
#pragma unroll
    for (int q = 0; q < 2; ++q) wf[t][q] = g.wpk2[((size_t)ct * (2 * kG2) + kh * kG2 + t) * 128 + q * 64 + lane];
  const f32x4 inv = *(const f32x4*)(g.scale2 + kC1 + c2), bias = *(const f32x4*)(g.bias2 + c2);
  const float refused = g.scale2[kC1 + kC2];

  const int npix2 = n2 * g.Wo2;  // of this workgroup
  // second layer: this lane's pixel of every tile, its window's first pixel (past the end: the last
  // pixel again, computed and stored again with the same bits)
  int abase[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int n = min(16 * m + lp, npix2 - 1);
    const int oy = n * g.rcp_wo2 >> 16, ox = n - oy * g.Wo2;
    abase[m] = 16 * ((oy * kS2 + kh * 2) * g.row_stride + (ox * kS2) * kP4 + lg);
  }

  // first layer: this lane's pixel of the wave's tile of a row (past the end: the last one again)
  const int ox1 = min(16 * ((wave >> 1) & 1) + lp, g.Wo1 - 1);
  int from[kCin];
#pragma unroll
  for (int s = 0; s < kCin; ++s) from[s] = (s * in_rows + 2 * lg) * kPitch + ox1 * kS1;
  const int to = 16 * ox1 * kP4 + 2 * c1;
  float minus_one = -1.0f;  // (opaque: a product by a known -1 becomes a conversion and a subtraction)
  asm volatile("" : "+v"(minus_one));

  // both halves of a frame's sums, bias, ReLU
  f32x4 own[OWN0];
  auto finish = [&](int b) __attribute__((always_inline)) {
    float* dst = g.out + ((size_t)b * g.Ho2 + row0) * g.Wo2 * kC2 + c2;
    const int m0 = kh == 0 ? 0 : OWN0;
#pragma unroll
    for (int m = 0; m < OWN0; ++m) {
      if (m == MT - OWN0 && kh != 0) break;
      const f32x4 other = sums[(ct * MT + m0 + m) * 64 + lane];
      const int n = min(16 * (m0 + m) + lp, npix2 - 1);
      f32x4 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = fmaxf(fmaf(own[m][e] + other[e], inv[e], bias[e]), 0.0f);
      *(f32x4*)(dst + (size_t)n * kC2) = r;
    }
  };

  store_frame();
  __syncthreads();
  if (!WHOLE) exchange_prepare(g.prep, (int)blockIdx.x * kNT + tid, (int)gridDim.x * kNT);
  int done = -1;  // the frame whose sums wait to be finished
  for (int b = first_frame; b < g.B; b += frame_step) {
    const bool more = WHOLE || b + frame_step < g.B;
    if (more) load_frame(min(b + frame_step, g.B - 1));  // (last round: a frame for no use)

    // (the last frame's outputs: half of the waves before the first layer, half behind it)
    if (kh != 0 && done >= 0) finish(done);

    // ---- first layer ----
    {
      i32x4 wd[kCin][3];
#pragma unroll
      for (int s = 0; s < kCin; ++s)
#pragma unroll
        for (int d = 0; d < 3; ++d) wd[s][d] = __builtin_bit_cast(i32x4, bank1[((half1 * kCin + s) * 3 + d) * 64 + lane]);
      const f32x4 s1 = *(const f32x4*)(affine1 + c1), b1 = *(const f32x4*)(affine1 + kC1 + c1);
      U2 rb[kCin][2];
      i32x4 even[3], odd[3];
      auto load_row = [&](int oy) __attribute__((always_inline)) {
        const int row = min(oy, n1 - 1) * (kS1 * kPitch);  // (past the end: the last row, for no use)
#pragma unroll
        for (int s = 0; s < kCin; ++s)
#pragma unroll
          for (int pp = 0; pp < 2; ++pp) rb[s][pp] = *(const U2*)(lds + from[s] + row + pp * kPitch);
      };
      auto multiply = [&](i32x4 (&a)[3]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kCin; ++s) {
          const i32x4 x = {(int)rb[s][0].x, (int)rb[s][0].y, (int)rb[s][1].x, (int)rb[s][1].y};
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            if (s == 0) a[d] = i32x4{0, 0, 0, 0};
            a[d] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wd[s][d], x, a[d], 0, 0, 0);
          }
        }
      };
      auto put = [&](const i32x4 (&a)[3], int oy) __attribute__((always_inline)) {
        u32x2 t0, t1;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          f32x2 r;
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int v = 2 * p + e;
            const float lo = (float)(__mul24(a[1][v], 254) + a[2][v]);  // (both sums are 192 * 128 * 127 at most)
            r[e] = fmaxf(fmaf(fmaf(lo, kInvRadix2, (float)a[0][v]), s1[v], b1[v]), 0.0f);
          }
          const f16x2 h = __builtin_convertvector(r, f16x2);
          const f32x2 rest = {fmaf((float)h[0], minus_one, r[0]), fmaf((float)h[1], minus_one, r[1])};
          t0[p] = __builtin_bit_cast(unsigned, h);
          t1[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(rest, f16x2));
        }
        uint8_t* at = image + (to + oy * g.row_stride * 16);
        *(u32x2*)at = t0;
        *(u32x2*)(at + 2 * kC1) = t1;
      };
      // a row's products run on the matrix pipe while the one before is scaled, split and stored
      auto mix = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
        }
      };
      int oy = kh;
      load_row(oy);
      multiply(even);
      load_row(oy + 2);
      for (;;) {
        multiply(odd);
        load_row(oy + 4);
        put(even, oy);
        mix();
        oy += 2;
        if (oy >= n1) break;
        multiply(even);
        load_row(oy + 4);
        put(odd, oy);
        mix();
        oy += 2;
        if (oy >= n1) break;
      }
    }
    if (kh == 0 && done >= 0) finish(done);
    __syncthreads();  // the image is complete, the frame's bytes are used up

    // ---- second layer ----
    {
      f32x4 acc[MT], low[MT];
      u32x4 x0[MT], x1[MT];
      auto tap = [&](int t) { return 16 * ((t / kK2) * g.row_stride + (t % kK2) * kP4); };
      auto mfma = [&](const u32x4& w, const u32x4& x, f32x4& c) __attribute__((always_inline)) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0, 0);
      };
#pragma unroll
      for (int m = 0; m < MT; ++m) x0[m] = *(const u32x4*)(image + abase[m]);
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        x1[m] = *(const u32x4*)(image + abase[m] + 2 * kC1);
        acc[m] = low[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
#pragma unroll
      for (int t = 0; t < kG2; ++t) {
        const int next = tap(t + 1);
        // (a term of the next tap is requested behind its last use; left alone, the scheduler sinks each
        // read to its use)
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          mfma(wf[t][1], x0[m], low[m]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          mfma(wf[t][0], x0[m], acc[m]);
          if (t + 1 < kG2) x0[m] = *(const u32x4*)(image + abase[m] + next);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          mfma(wf[t][0], x1[m], low[m]);
          if (t + 1 < kG2) x1[m] = *(const u32x4*)(image + abase[m] + next + 2 * kC1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m] += low[m];
      if (kh == 0) {
#pragma unroll
        for (int m = OWN0; m < MT; ++m) sums[(ct * MT + m) * 64 + lane] = acc[m];
#pragma unroll
        for (int m = 0; m < OWN0; ++m) own[m] = acc[m];
      } else {
#pragma unroll
        for (int m = 0; m < OWN0; ++m) sums[(ct * MT + m) * 64 + lane] = acc[m];
#pragma unroll
        for (int m = OWN0; m < MT; ++m) own[m - OWN0] = acc[m];
      }
    }
    if (more) store_frame();
    __syncthreads();  // the sums and the next frame's bytes are there, the image is used up
    asm volatile("" ::"s"(refused));  // (requested with the scales, here long since)
    done = b;
  }
  finish(done);
  // The host launches this kernel while the second layer's split is admitted; a graph recorded then may
  // run it after an update that is not, and gets that layer by its definition in fp32 (slow).
  if (__builtin_expect(refused != 0.0f, 0)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();  // the stores above are done
    const int8_t* digits = (const int8_t*)g.wpk1;
    for (int b = first_frame; b < g.B; b += frame_step) {
      const uint8_t* frame = g.obs + (size_t)b * ((size_t)kCin * g.H * g.W);
      float* mid = g.mid + (size_t)b * g.Ho1 * g.Wo1 * kC1;
      // (rows at a border of two workgroups: both write the same values)
      const int mid0 = kS2 * row0 * g.Wo1 * kC1;
#pragma unroll 1
      for (int i = mid0 + tid; i < mid0 + n1 * g.Wo1 * kC1; i += kNT) {
        const int n = i % kC1, pix = i / kC1, oy = pix / g.Wo1, ox = pix % g.Wo1;
        int d1 = 0, d2 = 0, d3 = 0;
#pragma unroll 1
        for (int k = 0; k < kCin * kK1 * kK1; ++k) {
          const int group = k / kK1, e = 8 * (group & 1) + k % kK1;
          const int x = frame[((size_t)(group / kK1) * g.H + oy * kS1 + group % kK1) * g.W + ox * kS1 + k % kK1] - 128;
          const int8_t* d = digits + 4 * ((((group / 4) * 3) * 4 + e / 4) * 64 + 32 * (group / 2 % 2) + n) + e % 4;
          d1 += x * d[0];
          d2 += x * d[4 * 4 * 64];
          d3 += x * d[2 * 4 * 4 * 64];
        }
        mid[i] = fmaxf(fmaf(fmaf((float)(d2 * 254 + d3), kInvRadix2, (float)d1), g.scale1[n], g.bias1[n]), 0.0f);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      const int out0 = row0 * g.Wo2 * kC2;
#pragma unroll 1
      for (int i = out0 + tid; i < out0 + npix2 * kC2; i += kNT) {
        const int n = i % kC2, pix = i / kC2, oy = pix / g.Wo2, ox = pix % g.Wo2;
        const float* x = mid + ((size_t)oy * kS2 * g.Wo1 + ox * kS2) * kC1;
        const float* w = g.w32 + (size_t)n * (kK2 * kK2 * kC1);
        float sum = 0.0f;
#pragma unroll 1
        for (int k = 0; k < kK2 * kK2 * kC1; ++k)
          sum = fmaf(x[(size_t)(k / (kK2 * kC1)) * g.Wo1 * kC1 + k % (kK2 * kC1)], w[k], sum);
        g.out[(size_t)b * g.Ho2 * g.Wo2 * kC2 + i] = fmaxf(sum + g.bias2[n], 0.0f);
      }
    }
  }
}

struct Layout {
  int row_stride, image_at, sums_at, bank_at;
  size_t bytes;
};
// The image's rows are padded so that output pixel n of the second layer reads piece 2 * kP4 * n +
// const modulo 16 also across the end of a row (no bank conflicts between the pixels of a tile); two
// rows of the byte frame lie 64 bytes apart modulo 256, so that the four lane groups of a tile (filter
// rows 2 lg, 2 lg + 1) read different banks.
Layout layout(int H, int Ho1, int Wo1, int Wo2) {
  Layout L;
  L.row_stride = Wo1 * kP4 + (((kP4 * Wo2 - Wo1 * kP4) % 8) + 8) % 8;
  L.image_at = kCin * H * kPitch;
  L.sums_at = L.image_at + 16 * Ho1 * L.row_stride;
  L.bank_at = L.sums_at + 16 * 4 * kMaxTiles * 64;
  L.bytes = (size_t)L.bank_at + 16 * 2 * kCin * 3 * 64 + 4 * 2 * kC1;
  return L;
}

}  // namespace

// Shapes: three byte planes, 8x8 / 4 -> 32 channels, then 4x4 / 2 -> 64 channels whose pixels fill
// seven tiles (frames of 72 x 128 and their like), no padding; whole 16-byte pieces in a frame row.
bool conv12_split_supported(int cin, int H, int W, const sf_conv& a, const sf_conv& b) {
  if (cin != kCin || a.k != kK1 || a.stride != kS1 || a.pad != 0 || a.cout != kC1) return false;
  if (b.k != kK2 || b.stride != kS2 || b.pad != 0 || b.cout != kC2) return false;
  if (W % 16 != 0 || W > kPitch || H < kK1 || W < kK1) return false;
  const int Ho1 = (H - kK1) / kS1 + 1, Wo1 = (W - kK1) / kS1 + 1;
  if (Ho1 < kK2 || Wo1 < kK2 || Wo1 > 32) return false;
  const int Ho2 = (Ho1 - kK2) / kS2 + 1, Wo2 = (Wo1 - kK2) / kS2 + 1, pieces = kCin * H * W / 16;
  if ((Ho2 * Wo2 + 15) / 16 != kMaxTiles || pieces > kNV * kNT) return false;
  if (Ho2 * Wo2 * Wo2 >= 65536 || pieces * (W / 16) >= 65536) return false;  // (reciprocal())
  return layout(H, Ho1, Wo1, Wo2).bytes <= kMaxLds;
}

// L1 on three digit planes, L2 on split operands; obs 4-byte aligned (the second layer's sums are this
// kernel's own: frames at any address have to come here); mid: room for L1's output, written by the
// fallback only; prep: see Args, marked as done if it is.
hipError_t launch_conv12_split(const ConvLayer& L1, const ConvLayer& L2, int B, const uint8_t* obs, float* mid, float* out,
                               ExchangePrep& prep, hipStream_t st) {
  if (B == 0) return hipSuccess;
  if (((uintptr_t)obs & 3) != 0 || L1.planes != 3 || (L2.Ho * L2.Wo + 15) / 16 != kMaxTiles) return hipErrorInvalidValue;
  const Layout L = layout(L1.H, L1.Ho, L1.Wo, L2.Wo);
  Args g;
  g.obs = obs; g.wpk1 = L1.ipk; g.scale1 = L1.spk; g.bias1 = L1.bpk8;
  g.wpk2 = (const u32x4*)L2.wsp; g.scale2 = L2.ssc; g.w32 = L2.wpk; g.bias2 = L2.bias; g.mid = mid; g.out = out;
  g.B = B; g.H = L1.H; g.W = L1.W; g.Ho1 = L1.Ho; g.Wo1 = L1.Wo; g.Ho2 = L2.Ho; g.Wo2 = L2.Wo;
  g.row_stride = L.row_stride; g.image_at = L.image_at; g.sums_at = L.sums_at; g.bank_at = L.bank_at;
  g.rcp_wo2 = reciprocal(L2.Wo); g.rcp_row = reciprocal(L1.W / 16);
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&] {
    for (const void* k : {(const void*)conv12_split_kernel<7>, (const void*)conv12_split_kernel<4>, (const void*)conv12_split_kernel<2>})
      if (attr_status == hipSuccess) attr_status = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
  });
  if (attr_status != hipSuccess) return attr_status;
  // Workgroups per frame.  A half takes 0.6 of a frame's time, a quarter 0.4: the fewest parts of the least
  // time over the rounds of 256 workgroups (a quarter up to 64 frames, a half up to 128 and from 257 to 384).
  const int limit[] = {0, 7, 4, 0, 2}, cost[] = {0, 10, 6, 0, 4};
  g.parts = 1;
  int blocks = B < 256 ? B : 256, least = (B + 255) / 256 * cost[1];
  for (int parts : {2, 4}) {
    const int items = B * parts, time = (items + 255) / 256 * cost[parts];
    if ((L2.Ho + parts - 1) / parts * L2.Wo > 16 * limit[parts] || time >= least) continue;
    g.parts = parts;
    blocks = items < 256 ? items : 256;
    least = time;
  }
  prep.done = g.parts > 1;
  g.prep = prep;
  auto kern = g.parts == 4 ? conv12_split_kernel<2> : g.parts == 2 ? conv12_split_kernel<4> : conv12_split_kernel<7>;
  kern<<<blocks, kNT, L.bytes, st>>>(g);
  return hipGetLastError();
}

}  // namespace sf
