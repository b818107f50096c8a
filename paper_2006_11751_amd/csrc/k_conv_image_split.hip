// Strided convolution of the plain encoder in fp32 configurations on the 16-bit matrix instructions
// (paper, App. "Model architectures": conv layers behind the first one), the frame's input image
// resident in LDS.
//
//   out[b][oy][ox][n] = act(bias[n] + sum_{p,q,c} in[b][oy*s + p][ox*s + q][c] * W[n][c][p][q])
//
// Arithmetic.  Scaled by powers of two, an activation is the sum of two fp16 numbers (11 + 11
// significant bits) and so is a weight; of the four products the three largest are kept: x0w1,
// x1w0, x0w0.  What is left out is at most 2^-21 of a product, 2^-23.8 root mean square, of random
// sign: less than what an fp32 accumulator is off after the 512 or 576 terms of these layers, and
// an accumulator here is rounded 3 times per 32 terms instead of 16 times: the result is nearer to
// the exact one.  That needs a sum that fp32 rounds often: with 16 taps other than zero the split is
// 1.5 times as far off as an fp32 sum in one piece, with one tap 2 to 5 times, with 128 of 512 0.6
// to 0.8 times, with all 0.4 times.  Banks with channels of few such roundings keep the fp32
// instructions (conv_image_split_pack).
// fp16 holds 2^-24 .. 65504, so every input channel has a scale of its own that takes the largest
// value it can have (a bound that follows from the weights of the layers before it, frames being
// bytes) into [2^14, 2^15], folded into the weights, and every output channel one that does the
// same for its largest folded weight.  Values are then exact to 22 bits from 2^-18 of the bound
// upward; below, the absolute error stays at 2^-40 of the bound.  Where that is not small against
// the rounding errors of the layer (a bound far above the values), the layer keeps the fp32 matrix
// instructions: the admission test of conv_image_split_pack.
//
// The tiled fp32 kernel (k_gemm_mfma.hip) was bound by the fp32 matrix instructions (1/16 of the
// rate) and staged every pixel once per window that covers it.  Here a workgroup of four waves
// walks rounds of FR frames: the image goes through registers, where it is scaled and split, into
// LDS, and after one barrier each wave computes 16 output channels of all pixels, its filter bank
// (both terms: 128 or 144 registers) resident.  Two workgroups share a CU, one loading while the
// other computes; or one of eight waves and two images does both at once (AHEAD).  Launch times: see
// launch_conv_image_split.
//
// v_mfma_f32_16x16x32_f16: lane l supplies A[i = l%16][k = 8*(l/16) + e] and B[k][j = l%16], e =
// 0..7 (16 bytes each); D[i][j] sits in lane j + 16*(i/4), register i%4.  A = weights (i = output
// channel), B = pixels: a lane ends up with four neighbouring channels of one pixel.  One
// instruction covers 32 input channels of one filter tap.
//
// LDS: a pixel is its CIN first terms, its CIN second terms and 16 bytes of padding (an odd number
// of 16-byte pieces); rows and frames are padded so that output pixel n of a round reads piece
// 2 * P4 * n + const modulo 16 also across the end of a row: neighbouring pixels two pieces apart,
// the four lane groups one, no bank conflicts.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "sf_internal.h"

namespace sf {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr size_t kMaxLds = 80 * 1024;  // two workgroups per CU

struct SplitArgs {
  const f32x4* in;      // [B][H][W][CIN]
  const u32x4* wpk;     // [N/16][G][2][64] lane operands, G = KS*KS*CIN/32
  const float* scale;   // [CIN] input scales, [N] inverse output scales, 1 if the split is not admitted
  const float* w32;     // [N][KS][KS][CIN]
  const float* bias;    // [N]
  float* out;           // [B][Ho*Wo][N]
  int B, H, W, Ho, Wo, N;
  int row_pad, frame_pad;  // 16-byte pieces appended to an image row / a frame in LDS
  int rcp_w, rcp_wo, rcp_npix;  // x / d = x * rcp >> 16, see reciprocal()
};
// ceil(65536 / d): exact for x * d < 65536
int reciprocal(int d) { return (65536 + d - 1) / d; }

// FR frames per round; their FR*Ho*Wo <= 16*MT output pixels form one row-major sequence of MT
// 16-pixel tiles, computed MP at a time.  NW: waves, 16 output channels each; NV: 16-byte pieces of a
// round's input per thread.  AHEAD: a CU's only workgroup, with two images in LDS: the pieces of the next round are
// fetched, scaled, split and stored between a round's products (four at a time: with more the registers of the
// filter bank spill, and a reload waits for the pieces).  A round takes 4.2 us, bound by the products and, over the
// chip, by the frames' 25 KB each.
template <int CIN, int KS, int FR, int MT, int MP, int NW, int NV, bool AHEAD>
__global__ __launch_bounds__(64 * NW, 2) void conv_image_split_kernel(SplitArgs g) {
  constexpr int kNT = 64 * NW;
  constexpr int STRIDE = 2;
  constexpr int C4 = CIN / 4;       // 16-byte pieces of a pixel in memory
  constexpr int C8 = CIN / 8;       // ... of one of its terms in LDS
  constexpr int P4 = 2 * C8 + 1;    // LDS pixel pitch in pieces
  constexpr int HALVES = CIN / 32;
  constexpr int G = KS * KS * HALVES;
  extern __shared__ __attribute__((aligned(16))) u32x4 img[];  // [FR][frame_stride] pieces

  static_assert(!AHEAD || (MT == MP && NV <= 8 && G >= 14), "one pass over the taps, with room for the pieces");
  static_assert(FR <= 2 && kNT % C4 == 0, "a thread's pieces: two frames at most, the same channels throughout");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lp = lane & 15, lg = lane >> 4;
  const int n0 = ((int)blockIdx.y * NW + wave) * 16;  // the wave's output channels
  const int npix = g.Ho * g.Wo;
  const int frame_pieces = g.H * g.W * C4;
  const int row_stride = g.W * P4 + g.row_pad;
  const int frame_stride = g.H * row_stride + g.frame_pad;

  u32x4 wf[G][2];
  auto load_bank = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
      for (int q = 0; q < 2; ++q) wf[t][q] = g.wpk[((size_t)(n0 / 16) * G + t) * 128 + q * 64 + lane];
  };
  if constexpr (!AHEAD) load_bank();
  const f32x4 scale = *(const f32x4*)(g.scale + (tid % C4) * 4);  // (a thread's pieces: the same channels)
  f32x4 inv, bias;
  if constexpr (!AHEAD) {
    inv = *(const f32x4*)(g.scale + CIN + n0 + 4 * lg);
    bias = *(const f32x4*)(g.bias + n0 + 4 * lg);
  }
  const float refused = g.scale[CIN + g.N];
  const int wave_n0 = __builtin_amdgcn_readfirstlane(n0);  // (kept in a scalar register for the fallback)

  // this lane's pixel of a tile: LDS piece of its window's first pixel (past the end: the last
  // pixel again, computed and stored again with the same bits)
  auto origin = [&](int m) {
    int n = 16 * m + lp;
    n = n < FR * npix ? n : FR * npix - 1;
    const int fr = FR == 1 ? 0 : n * g.rcp_npix >> 16, pix = n - fr * npix;
    const int oy = pix * g.rcp_wo >> 16, ox = pix - oy * g.Wo;
    return fr * frame_stride + (oy * STRIDE) * row_stride + (ox * STRIDE) * P4 + lg;
  };
  int abase[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) abase[m] = origin(m);

  const int n_rounds = (g.B + FR - 1) / FR;
  constexpr int NR = AHEAD ? 4 : NV;  // pieces in registers
  f32x4 v[NR];
  // piece u of a round
  // (opaque: computed ahead of the loop the places of all pieces would have to be spilled)
  auto thread = [&]() __attribute__((always_inline)) {
    int first = tid;
    asm volatile("" : "+v"(first));
    return first;
  };
  auto load = [&](int it, int u, int first) __attribute__((always_inline)) {
    // a last round with fewer frames re-reads its last piece instead of reading past the batch
    const uint8_t* src = (const uint8_t*)(g.in + (size_t)it * FR * frame_pieces);
    const uint32_t last = 16u * (uint32_t)(min(g.B - it * FR, FR) * frame_pieces - 1);
    v[u % NR] = *(const f32x4*)(src + min(16u * (uint32_t)(first + kNT * u), last));
  };
  auto put = [&](int u, u32x4* image, int first) __attribute__((always_inline)) {
    const int f = first + kNT * u;
    const bool second = FR == 2 && f >= frame_pieces;
    const int pix = (f - (second ? frame_pieces : 0)) / C4;
    int at = (second ? frame_stride : 0) + pix * P4 + (pix * g.rcp_w >> 16) * g.row_pad;
    at = min(at, FR * frame_stride);  // (past the end: a pixel behind the images, for no use)
    u32x2 t0, t1;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const f32x2 s = {v[u % NR][2 * p] * scale[2 * p], v[u % NR][2 * p + 1] * scale[2 * p + 1]};
      const f16x2 h = __builtin_convertvector(s, f16x2);
      const f32x2 rest = {fmaf((float)h[0], -1.0f, s[0]), fmaf((float)h[1], -1.0f, s[1])};
      t0[p] = __builtin_bit_cast(unsigned, h);
      t1[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(rest, f16x2));
    }
    u32x2* dst = (u32x2*)(image + at) + tid % C4;
    dst[0] = t0;
    dst[2 * C8] = t1;
  };
  if constexpr (AHEAD)
#pragma unroll
    for (int u = 0; u < NR; ++u) load(blockIdx.x, u, thread());
  if constexpr (AHEAD) load_bank();
  const int image_stride = FR * frame_stride + P4;
  f32x4* const affine = (f32x4*)(img + 2 * image_stride);  // AHEAD: [2][N / 4] inverse scales, biases
  if constexpr (AHEAD) {
    if (tid < g.N / 2) affine[tid] = ((const f32x4*)(tid < g.N / 4 ? g.scale + CIN : g.bias))[tid % (g.N / 4)];
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      put(u, img, thread());
      if (u + NR < NV) load(blockIdx.x, u + NR, thread());
    }
    __syncthreads();
  }
  int odd_round = 0;
  for (int it = blockIdx.x; it < n_rounds; it += gridDim.x) {
    const int frames = min(g.B - it * FR, FR), next_it = it + (int)gridDim.x;
    const u32x4* const image = img + (AHEAD && odd_round ? image_stride : 0);
    u32x4* const other = img + (AHEAD && odd_round ? 0 : image_stride);
    odd_round ^= 1;
    if constexpr (!AHEAD) {
      const int first = thread();
#pragma unroll
      for (int u = 0; u < NV; ++u) load(it, u, first);
#pragma unroll
      for (int u = 0; u < NV; ++u) put(u, img, first);
      __syncthreads();
    }
    asm volatile("" ::"s"(refused));  // (requested with the scales, here long since)

    float* dst = g.out + (size_t)it * FR * npix * g.N + n0 + 4 * lg;
    const int live = frames * npix;
    auto tap = [&](int t) {
      const int tp = t / HALVES, half = t % HALVES;
      return (tp / KS) * row_stride + (tp % KS) * P4 + 4 * half;
    };
    auto tiles = [&](auto m0c, auto mnc, auto morec) __attribute__((always_inline)) {
      constexpr bool MORE = decltype(morec)::value;
      constexpr int M0 = decltype(m0c)::value, MN = decltype(mnc)::value;
      // (the small products in an accumulator of their own: added to the large ones they would have
      // them rounded three times as often)
      f32x4 acc[MN], low[MN];
      u32x4 x0[MN], x1[MN];
#pragma unroll
      for (int m = 0; m < MN; ++m) {
        acc[m] = low[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        x0[m] = image[abase[M0 + m] + tap(0)];
        x1[m] = image[abase[M0 + m] + tap(0) + C8];
      }
      if constexpr (MORE)
#pragma unroll
        for (int u = 0; u < NR; ++u) load(next_it, u, thread());
#pragma unroll
      for (int t = 0; t < G; ++t) {
        const int next = tap(t + 1 < G ? t + 1 : t);
        auto mfma = [&](const u32x4& w, const u32x4& x, f32x4& c) __attribute__((always_inline)) {
          c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), c, 0, 0, 0);
        };
        if constexpr (AHEAD) {
          // a term of the next tap is requested behind its last use (left alone, the scheduler sinks each
          // read to its use)
#pragma unroll
          for (int m = 0; m < MN; ++m) {
            mfma(wf[t][1], x0[m], low[m]);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int m = 0; m < MN; ++m) {
            mfma(wf[t][0], x0[m], acc[m]);
            if (t + 1 < G) x0[m] = image[abase[M0 + m] + next];
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int m = 0; m < MN; ++m) {
            mfma(wf[t][0], x1[m], low[m]);
            if (t + 1 < G) x1[m] = image[abase[M0 + m] + next + C8];
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int m = 0; m < MN; ++m) {
            mfma(wf[t][1], x0[m], low[m]);
            mfma(wf[t][0], x0[m], acc[m]);
            mfma(wf[t][0], x1[m], low[m]);
            // the operands of the next tap, MN tiles ahead of their use
            if (t + 1 < G) {
              x0[m] = image[abase[M0 + m] + next];
              x1[m] = image[abase[M0 + m] + next + C8];
            }
            __builtin_amdgcn_sched_barrier(0);  // (left alone, the scheduler sinks each read to its use)
          }
        }
        if constexpr (MORE) {
          // the first pieces, asked for ahead of the taps, behind six of them, the others behind the last
          if (t >= 6 && t < 6 + NR) {
            put(t - 6, other, thread());
            if (t - 6 + NR < NV) load(next_it, t - 6 + NR, thread());
          }
          if (t >= G - (NV - NR)) put(t - (G - NV), other, thread());
        }
      }
      if constexpr (AHEAD) {
        inv = affine[(n0 >> 2) + lg];
        bias = affine[((g.N + n0) >> 2) + lg];
      }
#pragma unroll
      for (int m = 0; m < MN; ++m) {
        const int n = min(16 * (M0 + m) + lp, FR * npix - 1);
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = fmaxf(fmaf(acc[m][e] + low[m][e], inv[e], bias[e]), 0.0f);
        if (FR == 1 || n < live) *(f32x4*)(dst + (size_t)n * g.N) = r;
      }
    };
    using All = std::integral_constant<int, MP>;
    using Zero = std::integral_constant<int, 0>;
    if constexpr (AHEAD) {
      if (next_it < n_rounds)
        tiles(Zero{}, All{}, std::true_type{});
      else
        tiles(Zero{}, All{}, std::false_type{});
    } else {
      tiles(Zero{}, All{}, std::false_type{});
      if constexpr (MT > MP) tiles(All{}, std::integral_constant<int, MT - MP>{}, std::false_type{});
    }
    __syncthreads();  // every wave is done with this round's images
  }
  // The host launches this kernel while the split is admitted; a graph recorded then may run it after
  // an update that is not, and gets the layer by its definition in fp32 (slow, every wave its own
  // outputs once more).
  if (__builtin_expect(refused != 0.0f, 0)) {
    __syncthreads();
    const int fallback_lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    for (int it = blockIdx.x; it < n_rounds; it += gridDim.x) {
      const int todo = min(g.B - it * FR, FR) * npix * 16;
#pragma unroll 1
      for (int i = fallback_lane; i < todo; i += 64) {
        const int n = wave_n0 + (i & 15), at = i >> 4, fr = at / npix, pix = at % npix, oy = pix / g.Wo, ox = pix % g.Wo;
        const float* x = (const float*)g.in +
                         (((size_t)(it * FR + fr) * g.H + oy * STRIDE) * g.W + ox * STRIDE) * CIN;
        const float* w = g.w32 + (size_t)n * (KS * KS * CIN);
        float sum = 0.0f;
#pragma unroll 1
        for (int k = 0; k < KS * KS * CIN; ++k)
          sum = fmaf(x[(size_t)(k / (KS * CIN)) * g.W * CIN + k % (KS * CIN)], w[k], sum);
        g.out[((size_t)it * FR * npix + at) * g.N + n] = fmaxf(sum + g.bias[n], 0.0f);
      }
    }
  }
}

struct Layout {
  int row_pad, frame_pad;
  size_t lds_bytes;
};
Layout layout(int Cin, int FR, int H, int W, int Ho, int Wo) {
  const int P4 = Cin / 4 + 1;
  Layout L;
  L.row_pad = (((P4 * Wo - W * P4) % 8) + 8) % 8;
  const int row = W * P4 + L.row_pad;
  L.frame_pad = FR > 1 ? (((2 * P4 * Ho * Wo - H * row) % 16) + 16) % 16 : 0;
  L.lds_bytes = 16 * ((size_t)FR * (H * row + L.frame_pad) + P4);  // and a pixel that nobody reads
  return L;
}

// Which instantiation takes a layer: 0 none; 1: 4x4 on 32 channels, one frame per round in seven
// tiles; 2: 3x3 on 64 channels, two frames per round in three tiles (four frames in five tiles waste
// less of a tile, but leave room for one workgroup per CU).  The numbers of tiles, and of pieces per
// thread, are those of frames of 72 x 128 and their like, because a tile's place is a register and its
// loop is unrolled; nothing else stands against other frames, which need instantiations of their
// own (84 x 84: six and two tiles) and stay on k_gemm_mfma.hip, up to 2.7 times slower, without.
int variant(int Cin, int ksize, int stride, int pad, int H, int W, int N) {
  if (stride != 2 || pad != 0 || (N % 64) != 0 || H < ksize || W < ksize) return 0;
  const int Ho = (H - ksize) / 2 + 1, Wo = (W - ksize) / 2 + 1;
  if (17 * 256 / 8 * W >= 65536 || 128 * Ho * Wo >= 65536) return 0;  // (reciprocal())
  if (Cin == 32 && ksize == 4) {
    const int mt = (Ho * Wo + 15) / 16;
    if (mt == 7 && H * W * 8 <= 17 * 256 && layout(32, 1, H, W, Ho, Wo).lds_bytes <= kMaxLds) return 1;
  }
  if (Cin == 64 && ksize == 3)
    if (2 * Ho * Wo > 32 && 2 * Ho * Wo <= 48 && 2 * H * W * 16 <= 13 * 256 &&
        layout(64, 2, H, W, Ho, Wo).lds_bytes <= kMaxLds)
      return 2;
  return 0;
}

template <int CIN, int KS, int FR, int MT, int MP, int NW, int NV, bool AHEAD = false>
hipError_t launch_t(SplitArgs g, hipStream_t st) {
  const Layout L = layout(CIN, FR, g.H, g.W, g.Ho, g.Wo);
  g.row_pad = L.row_pad;
  g.frame_pad = L.frame_pad;
  g.rcp_w = reciprocal(g.W);
  g.rcp_wo = reciprocal(g.Wo);
  g.rcp_npix = reciprocal(g.Ho * g.Wo);
  auto kern = conv_image_split_kernel<CIN, KS, FR, MT, MP, NW, NV, AHEAD>;
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&] {
    attr_status = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)(AHEAD ? 2 * kMaxLds : kMaxLds));
  });
  if (attr_status != hipSuccess) return attr_status;
  const int n_rounds = (g.B + FR - 1) / FR, ny = g.N / (16 * NW);
  // eight waves per CU, each workgroup walking its share of the rounds
  const int per_chip = 2048 / NW, slots = ny >= per_chip ? 1 : per_chip / ny;
  const size_t lds = AHEAD ? 2 * L.lds_bytes + 8 * (size_t)g.N : L.lds_bytes;
  kern<<<dim3((unsigned)(n_rounds < slots ? n_rounds : slots), (unsigned)ny), 64 * NW, lds, st>>>(g);
  return hipGetLastError();
}

// Two images and the affine table in LDS, a vector of the table per thread.
bool ahead_fits(const SplitArgs& g) {
  return g.N % 128 == 0 && g.N <= 1024 &&
         2 * layout(64, 2, g.H, g.W, g.Ho, g.Wo).lds_bytes + 8 * (size_t)g.N <= 2 * kMaxLds;
}

// the power of two that takes v into [2^14, 2^15)
int power(double v) {
  if (!(v > 0.0 && v < 1e300)) return 0;
  int e;
  frexp(v, &e);  // v in [2^(e-1), 2^e)
  return e < -85 ? 100 : e > 115 ? -100 : 15 - e;
}

// Packing runs at every weight update: vectors over the input channels, and two builds of the loops, the
// second with the host's conversion instructions.
#define SF_INLINE inline __attribute__((always_inline))
#if defined(__HIP_DEVICE_COMPILE__) || !defined(__x86_64__)
#define SF_F16C
bool host_f16c() { return false; }
#else
#define SF_F16C __attribute__((target("avx2,f16c")))
bool host_f16c() { return __builtin_cpu_supports("avx2") && __builtin_cpu_supports("f16c"); }
#endif

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

struct Channel {
  double top;     // largest folded weight
  double spread;  // sum of |weight| * input bound
  double whole;   // sum of the mean squares of the terms
  double rounds;  // R of conv_image_split_pack
};

// The filter bank of an output channel as [tap][input channel], and what the admission test asks of it.
SF_INLINE Channel channel_loops(const float* wn, int cin, int kk, const double* fold, const double* bound,
                                const double* mean_sq, float* x) {
  for (int c = 0; c < cin; ++c)
    for (int t = 0; t < kk; ++t) x[(size_t)t * cin + c] = wn[(size_t)c * kk + t];
  auto vec = [](const double* v, int c) __attribute__((always_inline)) {
    f64x4 r;
    memcpy(&r, v + c, sizeof(r));
    return r;
  };
  auto size = [&](int t, int c) __attribute__((always_inline)) {
    f32x4 r;
    memcpy(&r, x + (size_t)t * cin + c, sizeof(r));
    return __builtin_convertvector(__builtin_elementwise_abs(r), f64x4);
  };
  auto sum = [](f64x4 v) __attribute__((always_inline)) { return (v[0] + v[1]) + (v[2] + v[3]); };
  f64x4 top = {0, 0, 0, 0}, spread = top, whole = top;
  for (int t = 0; t < kk; ++t)
    for (int c = 0; c < cin; c += 4) {
      const f64x4 v = size(t, c);
      top = __builtin_elementwise_max(top, v * vec(fold, c));
      spread += v * vec(bound, c);
      whole += v * v * vec(mean_sq, c);
    }
  Channel r{std::max(std::max(top[0], top[1]), std::max(top[2], top[3])), sum(spread), sum(whole), 0.0};
  // tap by tap: a tap's terms are seen by the later taps' roundings and half of its own
  double seen = 0.0, before = 0.0;
  const double least = 0x1p-40 * r.whole;
  for (int t = 0; t < kk; ++t) {
    f64x4 part = {0, 0, 0, 0}, roundings = part;
    for (int c = 0; c < cin; c += 4) {
      const f64x4 v = size(t, c), q = v * v * vec(mean_sq, c);
      part += q;
      roundings -= __builtin_convertvector(q >= least, f64x4);
    }
    const double own = sum(part);
    seen += sum(roundings) * (before + 0.5 * own);
    before += own;
  }
  r.rounds = seen / r.whole;
  return r;
}

// The same bank, scaled, in two terms.  (Two loops: from fp64 to fp16 without the stop there is no vector
// instruction.)
SF_INLINE void pack_loops(float* x, int n, int cin, int kk, const double* fold, double up, uint16_t* wpk) {
  const int halves = cin / 32, G = kk * halves;
  for (int t = 0; t < kk; ++t)
    for (int c = 0; c < cin; ++c) x[(size_t)t * cin + c] = (float)(x[(size_t)t * cin + c] * fold[c] * up);
  for (int gi = 0; gi < G; ++gi)
    for (int lg = 0; lg < 4; ++lg) {
      const int c = 32 * (gi % halves) + 8 * lg;
      f32x8 v;
      memcpy(&v, x + (size_t)(gi / halves) * cin + c, sizeof(v));
      const f16x8 h = __builtin_convertvector(v, f16x8);
      const f16x8 rest = __builtin_convertvector(v - __builtin_convertvector(h, f32x8), f16x8);
      uint16_t* at = wpk + ((((size_t)(n / 16) * G + gi) * 2) * 64 + lg * 16 + n % 16) * 8;
      memcpy(at, &h, sizeof(h));
      memcpy(at + 64 * 8, &rest, sizeof(rest));
    }
}
Channel channel_plain(const float* wn, int cin, int kk, const double* fold, const double* bound, const double* mean_sq,
                      float* x) {
  return channel_loops(wn, cin, kk, fold, bound, mean_sq, x);
}
SF_F16C Channel channel_f16c(const float* wn, int cin, int kk, const double* fold, const double* bound,
                             const double* mean_sq, float* x) {
  return channel_loops(wn, cin, kk, fold, bound, mean_sq, x);
}
void pack_plain(float* x, int n, int cin, int kk, const double* fold, double up, uint16_t* wpk) {
  pack_loops(x, n, cin, kk, fold, up, wpk);
}
SF_F16C void pack_f16c(float* x, int n, int cin, int kk, const double* fold, double up, uint16_t* wpk) {
  pack_loops(x, n, cin, kk, fold, up, wpk);
}

}  // namespace

bool conv_image_split_supported(int Cin, int ksize, int stride, int pad, int H, int W, int N) {
  return variant(Cin, ksize, stride, pad, H, W, N) != 0;
}

// Bound and mean square of every output channel of a ReLU'd convolution, from those of its input
// channels (w [cout][cin][k][k]; the mean square takes the terms of a sum as independent).
void conv_activation_range(const float* w, const float* bias, int cout, int cin, int k, std::vector<double>& bound,
                           std::vector<double>& mean_sq) {
  std::vector<double> b(cout), m(cout);
  for (int o = 0; o < cout; ++o) {
    double sb = fabs((double)bias[o]), sm = (double)bias[o] * bias[o];
    for (int c = 0; c < cin; ++c) {
      double l1 = 0.0, l2 = 0.0;
      for (int t = 0; t < k * k; ++t) {
        const double v = w[((size_t)o * cin + c) * k * k + t];
        l1 += fabs(v);
        l2 += v * v;
      }
      sb += l1 * bound[c];
      sm += l2 * mean_sq[c];
    }
    b[o] = sb;
    m[o] = sm;
  }
  bound.swap(b);
  mean_sq.swap(m);
}

// Weights in operand order, [N/16][G][2][64][8] fp16 bits: lane l of tap group gi holds, for e =
// 0..7, both terms of W[16 nt + l%16][c = 32 half + 8 (l/16) + e][p][q], gi = (p k + q)(cin/32) +
// half, times 2^(e_in[c]) and the output channel's scale; scale: [cin] input scales, [cout] inverse
// output scales, 0 or (not admitted) 1.  bound, mean_sq: of the input channels.
// Returns the admission ratio; the split runs where it is <= 1.  (Infinite or NaN bounds give a ratio
// that is not <= 1.)  With P_k the mean square of a channel's sum after k terms (in the order tap,
// input channel) and R = (sum of P_k over the terms that can round an accumulator: 2^-20 of the
// whole or more) / P_K, an fp32 sum is off by about sqrt(2 R) 2^-24 of its size (R = K / 2 where all taps are
// alike, 1 for a single tap).  The ratio is the largest over the channels of
//   - what the fixed part of the splitting errors can add up to, 2^-40 of an input bound and 2^-39
//     of the largest folded weight, over that error;
//   - 192 / R: what is left out of the products is proportional to the sum's size, so it has to be
//     rounded often to be as far off in fp32.  Error of the new state against 64 bits, split over
//     fp32 kernel, 64 hidden units, R of 230 and more (random weights: normal, Laplace, uniform): 0.80
//     to 0.84 where k_gemm_mfma.hip takes K in one piece (handles for 1100 rows), 0.93 to 0.99 in two
//     pieces (400 rows), 0.99 to 1.06 in four (64 rows); R = 160: 0.93, 1.04, 1.09.
double conv_image_split_pack(const float* w, int cout, int cin, int k, const std::vector<double>& bound,
                             const std::vector<double>& mean_sq, std::vector<uint16_t>& wpk, std::vector<float>& scale) {
  constexpr double kRounds = 192.0;
  const int kk = k * k, K = cin * kk;
  wpk.assign((size_t)cout * K * 2, 0);
  scale.assign(cin + cout + 1, 1.0f);
  std::vector<double> fold(cin);  // 1 / input scale
  double worst = 0.0;
  for (int c = 0; c < cin; ++c) {
    const int e = power(bound[c]);
    scale[c] = (float)ldexp(1.0, e);
    fold[c] = ldexp(1.0, -e);
    if (!(bound[c] < 1e30)) worst = INFINITY;
  }
  std::vector<float> x(K);
  const bool f16c = host_f16c();
  for (int n = 0; n < cout; ++n) {
    const Channel ch = (f16c ? channel_f16c : channel_plain)(w + (size_t)n * K, cin, kk, fold.data(), bound.data(),
                                                            mean_sq.data(), x.data());
    const int e = power(ch.top);
    const double up = ldexp(1.0, e);
    scale[cin + n] = (float)ldexp(1.0, -e);
    // folded weights have an absolute error of 2^-25 at a largest value of 2^14 or more; an input
    // of scaled size 2^15 multiplies it
    const double fixed = ldexp(ch.spread, -40) + K * ldexp(1.0, 15 - 25 - e);
    const double ref = sqrt(2.0 * ch.rounds) * ldexp(1.0, -24) * sqrt(ch.whole);
    // (a channel without weights has nothing to get wrong)
    if (ch.top > 0.0) worst = std::max(worst, ref > 0.0 ? std::max(fixed / ref, kRounds / ch.rounds) : INFINITY);
    (f16c ? pack_f16c : pack_plain)(x.data(), n, cin, kk, fold.data(), up, wpk.data());
  }
  scale[cin + cout] = worst <= 1.0 ? 0.0f : 1.0f;
  return worst;
}

// in [B][H][W][Cin] fp32; w32 the fp32 weights [N][k][k][Cin] -> out [B][Ho*Wo][N] fp32, ReLU'd.
// Launch times (us) against k_gemm_mfma.hip, conv2 / conv3 of the standard network: 16 rows 6.8 / 4.7
// (7.2 / 7.6), 333 rows 13.7 / 9.2 (26 / 16), 1024 rows 27 / 15 (72 / 34), 2048 rows 50 / 26
// (126 / 57).  At 1024 rows conv2 reads 70 MB and writes 26: 3.5 TB/s.
hipError_t launch_conv_image_split(const float* in, const uint16_t* wpk, const float* scale, const float* w32,
                                   const float* bias, float* out, int B, int H, int W, int Cin, int ksize, int N, hipStream_t st) {
  if (B == 0) return hipSuccess;
  SplitArgs g;
  g.in = (const f32x4*)in; g.wpk = (const u32x4*)wpk; g.scale = scale; g.w32 = w32; g.bias = bias; g.out = out;
  g.B = B; g.H = H; g.W = W; g.Ho = (H - ksize) / 2 + 1; g.Wo = (W - ksize) / 2 + 1; g.N = N;
  g.row_pad = g.frame_pad = 0;
  switch (variant(Cin, ksize, 2, 0, H, W, N)) {
    case 1: return launch_t<32, 4, 1, 7, 4, 4, 17>(g, st);
    case 2:
      // few frames: one per round and two waves, so that a CU has half of the filter bank to fetch (16 rows
      // 5.6 -> 4.0 us; beyond 256 workgroups no faster: whole steps at 128 / 256 rows 38.2, 37.6 / 45.4, 46.9)
      if ((long long)B * (N / 32) <= 256) return launch_t<64, 3, 1, 2, 2, 2, 13>(g, st);
      // From half the chip in workgroups of eight waves to a second round of few of them: the next round on the way
      // under this one's products.  Steps of the standard network at 128 output channels, us, without / with:
      // 258 rows 53.7 / 53.3, 400 rows 57.0 / 56.6, 512 rows 62.0 / 61.1, 514 rows 82.0 / 78.7, 640 rows 83.7 / 82.4,
      // 768 rows 87.7 / 87.5, 896 rows 93.6 / 95.2, 1500 rows 142 / 147.  (A measured window, without a cause: alone the
      // kernel is the faster one beyond it, too, 2048 rows 25 / 23, but the launches around it get longer there, which
      // has not been explained.  Below 256 rows it is not faster, 200 rows 6.0 / 7.6.)
      if (const long long work = (long long)((B + 1) / 2) * (N / 128); ahead_fits(g) && work > 128 && work <= 320)
        return launch_t<64, 3, 2, 3, 3, 8, 7, true>(g, st);
      return launch_t<64, 3, 2, 3, 3, 4, 13>(g, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sf
