// First and second convolution of the plain encoder in bf16 configurations as one kernel
// (paper, App. "Model architectures": the convolutional encoder), so that the first layer's
// output (the largest tensor of the step: 17 x 31 x 32 values per frame) never leaves the
// compute unit.  Run as two launches, the first layer writes 138 MB at B = 4096 and the second
// reads them straight back: 45 % of the step's HBM traffic.
//
// A workgroup of eight waves, one per CU, walks frames b, b + gridDim.x, ...  Between two barriers
// it computes the second layer of one frame and the first layer of the next, into two LDS images in
// turn; half of the waves take the first layer first, the other half the second, so that each SIMD
// has one wave on either: the first layer's vector instructions (scaling, ReLU, rounding) run beside
// the second's matrix instructions.
//   first layer, 8x8 / 4 -> 32 channels, on the int8 MFMA against the fixed-point digit planes of its
//     filter bank (two planes; see k_conv1_i8.hip for the arithmetic): the planar byte frame lies in LDS
//     as byte - 128; a wave takes 16 channels of half of a row's pixels, every second row; its bf16
//     results go into a channels-last image (pixel pitch 64 + 16 bytes, rows padded: the layout of
//     k_conv_image_bf16.hip).  Weights as the A operand leave four neighbouring channels of a pixel in a
//     lane: one 8-byte LDS write.
//   second layer, 4x4 / 2 -> 64 channels, on v_mfma_f32_16x16x32_bf16 out of that image: a wave owns 16
//     channels of four or three of the seven 16-pixel tiles; bias, ReLU, bf16, one 8-byte store of four
//     channels per lane and tile.
// Both banks stay in registers.  The sums, epilogues and roundings are those of the two separate
// kernels, so the results are the same bits.
//
// v_mfma_i32_16x16x64_i8: lane l supplies 16 bytes of A[i = l%16] and of B[j = l%16], the k block l/16;
// v_mfma_f32_16x16x32_bf16: A[i = l%16][k = 8*(l/16) + e], B[k][j = l%16]; both: D[i][j] sits in lane
// j + 16*(i/4), register i%4.
#include <mutex>
#include <type_traits>

#include "sf_internal.h"

namespace sf {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kNT = 512;
constexpr int kCin = 3, kK1 = 8, kS1 = 4, kC1 = 32;  // first layer: planes, filter, stride, channels
constexpr int kK2 = 4, kS2 = 2, kC2 = 64;            // second layer: filter, stride, channels
constexpr int kMaxTiles = 7;                         // 16-pixel tiles of the second layer
constexpr int kP4 = kC1 / 8 + 1;                     // LDS pixel pitch of the image in 16-byte pieces
constexpr int kNV = 4;                               // 16-byte pieces of a byte frame per thread
constexpr int kG2 = kK2 * kK2;                       // filter taps of the second layer
constexpr int kPitch = 160;                          // byte-frame row in LDS
constexpr size_t kMaxLds = 160 * 1024;
constexpr float kInvRadix = 1.0f / 254.0f;

struct __attribute__((packed, aligned(4))) U2 {
  uint32_t x, y;
};

struct Conv12Args {
  const uint8_t* obs;   // [B][3][H][W] bytes
  const int* wpk1;      // digit planes of the first filter bank, lane order of k_conv1_i8.hip
  const float* scale1;  // [32]
  const float* bias1;   // [32]
  const u32x4* wpk2;    // [4][16][64] lane fragments of the second filter bank
  const float* bias2;   // [64]
  uint16_t* out;        // bf16 [B][Ho2*Wo2][64]
  int B, H, W, Ho1, Wo1, Ho2, Wo2;
  int row_stride;       // image row pitch in pieces
  int image_at;         // LDS offset of the two images
  int rcp_wo2, rcp_row; // x / d = x * rcp >> 16 for Wo2, W / 16
  int parts;            // workgroups per frame
  ExchangePrep prep;    // with several workgroups per frame: work for a later launch (sf_exchange.h)
};

int reciprocal(int d) { return (65536 + d - 1) / d; }  // exact for x * d < 65536

// FLAT: the byte frame lies in LDS as in memory; otherwise (rows of whole 16-byte pieces) its rows are
// kPitch bytes apart: two of them 64 bytes modulo 256, so that the four lane groups of a tile (filter
// rows 2 lg, 2 lg + 1) read different banks, and at offsets known to the compiler.
// MT: 16-pixel tiles of the second layer per workgroup.  Few frames are dealt to two or four workgroups
// each, by rows of the second layer's output (the first layer's rows at a border are computed twice), with
// MT = 4 or 2 tiles.
template <bool FLAT, int MT>
__global__ __launch_bounds__(kNT, 2) void conv12_fused_bf16_kernel(Conv12Args g) {
  constexpr bool WHOLE = MT == kMaxTiles;
  constexpr int TILES = (MT + 1) / 2;  // of the first half of the waves
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lp = lane & 15, lg = lane >> 4;
  const int half1 = wave & 1;               // first layer: channel half
  const int ct = wave & 3, hi = wave >> 2;  // second layer: channel tile, first or last pixel tiles
  const int pitch = FLAT ? g.W : kPitch;

  // rows [row0, row0 + n2) of the second layer's output, n1 of the first layer's, in_rows of the image
  const int part = WHOLE ? 0 : (int)blockIdx.x % g.parts;
  const int row0 = WHOLE ? 0 : part * g.Ho2 / g.parts;
  const int n2 = WHOLE ? g.Ho2 : (part + 1) * g.Ho2 / g.parts - row0;
  const int n1 = WHOLE ? g.Ho1 : kS2 * (n2 - 1) + kK2;
  const int in_rows = WHOLE ? g.H : kS1 * (n1 - 1) + kK1;
  const int first_frame = WHOLE ? (int)blockIdx.x : (int)blockIdx.x / g.parts;
  const int stride = WHOLE ? (int)gridDim.x : (int)gridDim.x / g.parts;  // (the same part of every frame)

  const int row_pieces = g.W >> 4, pieces = WHOLE ? kCin * g.H * g.W / 16 : kCin * in_rows * row_pieces;
  u32x4 fv[kNV];
  auto load_frame = [&](int b) {
    const uint8_t* src = g.obs + (size_t)b * ((size_t)kCin * g.H * g.W);
#pragma unroll
    for (int u = 0; u < kNV; ++u) {
      const int f = min(tid + kNT * u, pieces - 1);
      uint32_t at = 16u * (uint32_t)f;
      if (!WHOLE) {
        const int plane = (f >= in_rows * row_pieces) + (f >= 2 * in_rows * row_pieces);
        at += (uint32_t)((plane * (g.H - in_rows) + kS1 * kS2 * row0) * g.W);
      }
      fv[u] = *(const u32x4*)(src + at);
    }
  };
  auto store_frame = [&]() {
#pragma unroll
    for (int u = 0; u < kNV; ++u) {
      const int f = min(tid + kNT * u, pieces - 1);
      int at = 16 * f;
      if (!FLAT) {
        const int row = f * g.rcp_row >> 16;
        at += row * (kPitch - g.W);
      }
      *(u32x4*)(lds + at) = fv[u] ^ 0x80808080u;
    }
  };
  load_frame(first_frame);

  // ---- operands that stay in registers ----
  i32x4 wd[kCin][2];
#pragma unroll
  for (int s = 0; s < kCin; ++s)
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int w = 0; w < 4; ++w)
        wd[s][d][w] = g.wpk1[(((2 * s + (lg >> 1)) * 3 + d) * 4 + w) * 64 + 32 * (lg & 1) + 16 * half1 + lp];
  const int c1 = 16 * half1 + 4 * lg, c2 = 16 * ct + 4 * lg;  // this lane's four channels
  const f32x4 s1 = *(const f32x4*)(g.scale1 + c1), b1 = *(const f32x4*)(g.bias1 + c1);
  u32x4 wf[kG2];
#pragma unroll
  for (int t = 0; t < kG2; ++t) wf[t] = g.wpk2[((size_t)ct * kG2 + t) * 64 + lane];
  const f32x4 bias = *(const f32x4*)(g.bias2 + c2);

  // first layer: this lane's pixel of the wave's tile of a row (past the end: the last one again)
  const int ox1 = min(16 * ((wave >> 1) & 1) + lp, g.Wo1 - 1);
  int from[kCin];
#pragma unroll
  for (int s = 0; s < kCin; ++s) from[s] = (s * in_rows + 2 * lg) * pitch + ox1 * kS1;
  const int to = 16 * ox1 * kP4 + 2 * c1;
  // second layer: this lane's pixel of the wave's tiles, its window's first pixel (past the end: the last
  // pixel again, computed and stored again with the same bits)
  const int npix2 = n2 * g.Wo2;
  auto pixel = [&](int m) { return min(16 * (TILES * hi + m) + lp, npix2 - 1); };
  int abase[TILES];
#pragma unroll
  for (int m = 0; m < TILES; ++m) {
    const int n = pixel(m), oy = n * g.rcp_wo2 >> 16, ox = n - oy * g.Wo2;
    abase[m] = 16 * ((oy * kS2) * g.row_stride + (ox * kS2) * kP4 + lg);
  }
  const int image_bytes = 16 * g.Ho1 * g.row_stride;

  auto first_layer = [&](uint8_t* image) __attribute__((always_inline)) {
    U2 rb[kCin][2];
    i32x4 even[2], odd[2];
    auto load_row = [&](int oy) __attribute__((always_inline)) {
      const int row = min(oy, n1 - 1) * (kS1 * pitch);  // (past the end: the last row, for no use)
#pragma unroll
      for (int s = 0; s < kCin; ++s)
#pragma unroll
        for (int pp = 0; pp < 2; ++pp) rb[s][pp] = *(const U2*)(lds + from[s] + row + pp * pitch);
    };
    auto multiply = [&](i32x4 (&a)[2]) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < kCin; ++s) {
        const i32x4 x = {(int)rb[s][0].x, (int)rb[s][0].y, (int)rb[s][1].x, (int)rb[s][1].y};
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          if (s == 0) a[d] = i32x4{0, 0, 0, 0};
          a[d] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wd[s][d], x, a[d], 0, 0, 0);
        }
      }
    };
    auto put = [&](const i32x4 (&a)[2], int oy) __attribute__((always_inline)) {
      u32x2 t;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        f32x2 r;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int v = 2 * p + e;
          r[e] = fmaxf(fmaf(fmaf((float)a[1][v], kInvRadix, (float)a[0][v]), s1[v], b1[v]), 0.0f);
        }
        t[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(r, bf16x2));
      }
      *(u32x2*)(image + (to + oy * g.row_stride * 16)) = t;
    };
    // a row's products run on the matrix pipe while the one before is scaled, rounded and stored
    int oy = hi;
    load_row(oy);
    multiply(even);
    load_row(oy + 2);
    for (;;) {
      multiply(odd);
      load_row(oy + 4);
      put(even, oy);
      oy += 2;
      if (oy >= n1) break;
      multiply(even);
      load_row(oy + 4);
      put(odd, oy);
      oy += 2;
      if (oy >= n1) break;
    }
  };

  auto second_layer = [&](const uint8_t* image, int b) __attribute__((always_inline)) {
    auto tiles = [&](auto mnc) __attribute__((always_inline)) {
      constexpr int MN = decltype(mnc)::value;
      f32x4 acc[MN];
      u32x4 x[2][MN];  // two taps in flight
      auto load_tap = [&](int t, int m) __attribute__((always_inline)) {
        x[t & 1][m] = *(const u32x4*)(image + (abase[m] + 16 * ((t / kK2) * g.row_stride + (t % kK2) * kP4)));
      };
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int m = 0; m < MN; ++m) load_tap(t, m);
#pragma unroll
      for (int m = 0; m < MN; ++m) acc[m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int t = 0; t < kG2; ++t)
#pragma unroll
        for (int m = 0; m < MN; ++m) {
          acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[t]),
                                                           __builtin_bit_cast(bf16x8, x[t & 1][m]), acc[m], 0, 0, 0);
          if (t + 2 < kG2) load_tap(t + 2, m);
          __builtin_amdgcn_sched_barrier(0);  // (left alone, the scheduler sinks each read to its use)
        }
      uint8_t* dst = (uint8_t*)g.out + ((size_t)b * g.Ho2 + row0) * g.Wo2 * (2 * kC2);
#pragma unroll
      for (int m = 0; m < MN; ++m) {
        float r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = fmaxf(acc[m][e] + bias[e], 0.0f);
        const f32x2 lo = {r[0], r[1]}, up = {r[2], r[3]};
        u32x2 o;
        o[0] = __builtin_bit_cast(unsigned, __builtin_convertvector(lo, bf16x2));
        o[1] = __builtin_bit_cast(unsigned, __builtin_convertvector(up, bf16x2));
        *(u32x2*)(dst + (uint32_t)(pixel(m) * (2 * kC2) + 2 * c2)) = o;
      }
    };
    if (hi)
      tiles(std::integral_constant<int, MT - TILES>{});
    else
      tiles(std::integral_constant<int, TILES>{});
  };

  uint8_t* image = lds + g.image_at;        // of the frame whose second layer is next
  uint8_t* other = image + image_bytes;
  int b = first_frame;
  store_frame();
  __syncthreads();
  if (!WHOLE) exchange_prepare(g.prep, (int)blockIdx.x * kNT + tid, (int)gridDim.x * kNT);
  if (WHOLE || b + stride < g.B) load_frame(min(b + stride, g.B - 1));  // (no frame left: one for no use)
  first_layer(image);
  __syncthreads();
  if (WHOLE || b + stride < g.B) {
    store_frame();
    __syncthreads();
  }
  for (; b < g.B; b += stride) {
    const bool more = b + stride < g.B;
    if (WHOLE || more) load_frame(min(b + 2 * stride, g.B - 1));
#pragma unroll 1
    for (int turn = 0; turn < 2; ++turn) {
      if (turn == hi) {
        if (more) first_layer(other);
      } else {
        second_layer(image, b);
      }
    }
    if (!WHOLE && !more) break;
    __syncthreads();  // one image is used up, the other complete; the frame's bytes are used up
    store_frame();
    __syncthreads();
    uint8_t* t = image;
    image = other;
    other = t;
  }
}

// Image row pitch in pieces: congruent to kP4 * Wo2 modulo 8 (then output pixel n of the second layer reads
// piece 2 * kP4 * n + const modulo 16 also across the end of an output row: no bank conflicts between the 16
// pixels of a tile).
int image_row_stride(int Wo1, int Wo2) {
  int r = Wo1 * kP4;
  while (r % 8 != (kP4 * Wo2) % 8) ++r;
  return r;
}
bool flat(int W) { return W % 16 != 0 || W > kPitch; }
int frame_lds_bytes(int H, int W) { return kCin * H * (flat(W) ? W : kPitch); }

}  // namespace

// Shapes: three byte planes, first layer 8x8 / 4 -> 32 channels with at most 32 pixels per output row,
// second layer 4x4 / 2 -> 64 channels with seven 16-pixel tiles, both without padding and with ReLU; frame a
// multiple of 16 bytes.
bool conv12_fused_bf16_supported(int cin, int H, int W, const sf_conv& c1, const sf_conv& c2) {
  if (cin != kCin || c1.k != kK1 || c1.stride != kS1 || c1.pad != 0 || c1.cout != kC1) return false;
  if (c2.k != kK2 || c2.stride != kS2 || c2.pad != 0 || c2.cout != kC2) return false;
  if (W % 4 != 0 || H < kK1 || W < kK1) return false;
  const int Ho1 = (H - kK1) / kS1 + 1, Wo1 = (W - kK1) / kS1 + 1;
  if (Wo1 > 32 || Ho1 < kK2 || Wo1 < kK2) return false;
  const int Ho2 = (Ho1 - kK2) / kS2 + 1, Wo2 = (Wo1 - kK2) / kS2 + 1;
  // seven 16-pixel tiles
  if ((Ho2 * Wo2 + 15) / 16 != kMaxTiles) return false;
  const int frame_bytes = cin * H * W;
  if (frame_bytes % 16 != 0 || frame_bytes > kNV * kNT * 16) return false;
  if (Ho2 * Wo2 * Wo2 >= 65536 || frame_bytes / 16 * (W / 16) >= 65536) return false;  // (reciprocal())
  return frame_lds_bytes(H, W) + 2 * 16 * (size_t)Ho1 * image_row_stride(Wo1, Wo2) <= kMaxLds;
}

// L1, L2: the two layers as executed separately (L1's digit planes, scales and bias, L2's
// image-kernel fragments and bias); out: bf16 [B][Ho2*Wo2][64].
hipError_t launch_conv12_fused_bf16(const ConvLayer& L1, const ConvLayer& L2, int B, const uint8_t* obs,
                                    void* out, ExchangePrep& prep, hipStream_t st) {
  if (B == 0) return hipSuccess;
  if (((uintptr_t)obs & 15) != 0 || L1.planes != 2 || (L2.Ho * L2.Wo + 15) / 16 != kMaxTiles) return hipErrorInvalidValue;
  Conv12Args g;
  g.obs = obs; g.wpk1 = L1.ipk; g.scale1 = L1.spk; g.bias1 = L1.bpk8;
  g.wpk2 = (const u32x4*)L2.wbf; g.bias2 = L2.bbf; g.out = (uint16_t*)out;
  g.B = B; g.H = L1.H; g.W = L1.W; g.Ho1 = L1.Ho; g.Wo1 = L1.Wo; g.Ho2 = L2.Ho; g.Wo2 = L2.Wo;
  g.row_stride = image_row_stride(L1.Wo, L2.Wo);
  g.image_at = (frame_lds_bytes(L1.H, L1.W) + 15) & ~15;
  g.rcp_wo2 = reciprocal(L2.Wo); g.rcp_row = L1.W >= 16 ? reciprocal(L1.W / 16) : 0;
  const size_t lds = (size_t)g.image_at + 2 * 16 * (size_t)L1.Ho * g.row_stride;
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&] {
    for (const void* k : {(const void*)conv12_fused_bf16_kernel<true, 7>, (const void*)conv12_fused_bf16_kernel<false, 7>,
                          (const void*)conv12_fused_bf16_kernel<false, 4>, (const void*)conv12_fused_bf16_kernel<false, 2>})
      if (attr_status == hipSuccess) attr_status = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
  });
  if (attr_status != hipSuccess) return attr_status;
  // Workgroups per frame: as many as run at once (one per CU), rows of whole 16-byte pieces.
  auto fits = [&](int parts, int tiles) {
    return !flat(L1.W) && B * parts <= 256 && (L2.Ho + parts - 1) / parts * L2.Wo <= 16 * tiles;
  };
  g.parts = fits(4, 2) ? 4 : fits(2, 4) ? 2 : 1;
  prep.done = g.parts > 1;
  g.prep = prep;
  auto kern = flat(L1.W) ? conv12_fused_bf16_kernel<true, 7>
              : g.parts == 4 ? conv12_fused_bf16_kernel<false, 2>
              : g.parts == 2 ? conv12_fused_bf16_kernel<false, 4>
                             : conv12_fused_bf16_kernel<false, 7>;
  kern<<<g.parts > 1 ? B * g.parts : B < 256 ? B : 256, kNT, lds, st>>>(g);
  return hipGetLastError();
}

}  // namespace sf
