// FC layer of 16-bit configurations on many rows (paper, App. "Model architectures": the layer behind the
// convolutional and the residual encoder):
//   out[m][n] = relu(bias[n] + sum_k x[m][k] * w[n][k]),  x and w bf16 or (F16) fp16, fp32 accumulation.
//
// What bounds it: 128 rows x 64 units per workgroup fill the chip in one round (4096 x 512, 8192 x 256) and
// leave each CU 24 KB per 64 numbers of K to fetch and 256 cycles of products, so that the time is how much is
// under way: with two chunks ahead in registers (k_conv_bf16.hip) a chunk took 1.5 k cycles, most of them
// the trip of activations that another XCD wrote.  Here a ring of kDepth chunks in LDS is filled by loads
// that go there directly (no registers, no LDS store instructions): all but two of them are on their way.
// One barrier per two chunks: it says that they have come and that the two before them have been read (one
// per chunk: 2 % slower at 4096 rows).  Medians of a kernel trace: 2304 -> 512 in bf16 at 4096 rows 24.4 -> 18.7 us
// (12.1 TB/s out of the L2s), 4608 -> 256 in fp16 at 8192 rows 45.1 -> 37.8.
//
// A load instruction writes 64 x 16 bytes in lane order, so rows (128 bytes) have no padding; instead the
// 16-byte pieces of a row are exchanged by the row's number, on the side of the source: slot s of row r holds
// piece s ^ (r / 2 % 8), and 16 neighbouring rows read different banks.
//
// The waits are counted by hand: the compiler takes every LDS read behind such a load for dependent on it and
// would wait for all of them, so the reads are written as assembly (with their own wait in the same block).
//
// Tiles of 32 x 32 per wave, K in order in one accumulator, as in k_conv_bf16.hip: the same bits,
// whatever the tile of the workgroup.
#include <mutex>

#include "sf_internal.h"

namespace sf {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) unsigned char LdsByte;

constexpr int kBN = 64;      // units per workgroup
constexpr int kRow = 128;    // bytes of a chunk's row: 64 numbers
constexpr int kMaxLds = 160 * 1024;

struct Fc16Args {
  const uint8_t* x;    // [M][K]
  const uint8_t* w;    // [N][K]
  const float* bias;   // [N]
  void* out;           // [M][N]
  int M, N, K;
};

template <int BM>
constexpr int chunk_bytes() { return (BM + kBN) * kRow; }
template <int BM>
constexpr int depth() { return 144 * 1024 / chunk_bytes<BM>() / 2 * 2; }  // 6 (128 rows), 8, 12

// 16 bytes per lane to LDS, in lane order (a function of its own: the host pass knows no such size)
__device__ __attribute__((always_inline)) inline void load_lds(__amdgpu_buffer_rsrc_t from, LdsByte* to, int at, int k) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, to, 16, at, k, 0, 0);
}

// BM rows per workgroup, 32 x 32 per wave.
template <int BM, bool F16, bool OUT_BF16>
__global__ __launch_bounds__(4 * BM, 2) void fc16_kernel(Fc16Args g) {
  constexpr int NW = BM / 16, kDepth = depth<BM>(), CH = chunk_bytes<BM>();
  constexpr int L = CH / 1024 / NW;  // load instructions of a wave per chunk
  static_assert(2 * NW == BM / 8 && L * NW * 1024 == CH && (kDepth - 4) * L < 64, "whole instructions, as many as the counter holds");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, lh = lane >> 5;
  const int rt = wave >> 1, ct = wave & 1;  // the wave's 32 rows, 32 units

  // tiles in runs of neighbours per XCD: the units of a row tile read the same rows out of its L2
  const int n_ct = g.N / kBN, n_tiles = (g.M + BM - 1) / BM * n_ct, per_xcd = (n_tiles + 7) / 8;
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (tile >= n_tiles) return;
  const int m0 = tile / n_ct * BM, n0 = tile % n_ct * kBN;
  const int rows = min(g.M - m0, BM);

  const int pitch = 2 * g.K, n_chunks = g.K / 64;
  const auto xs = __builtin_amdgcn_make_buffer_rsrc((void*)(g.x + (size_t)m0 * pitch), 0, rows * pitch, 0x00027000);
  const auto ws = __builtin_amdgcn_make_buffer_rsrc((void*)(g.w + (size_t)n0 * pitch), 0, kBN * pitch, 0x00027000);

  f32x4 bias[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) bias[q] = *(const f32x4*)(g.bias + n0 + 32 * ct + 8 * q + 4 * lh);

  // load instruction j of this wave: eight rows, of x (j < 2: BM / 8 instructions of NW waves), then of w (past the
  // last row: that row again, never stored)
  int at[L];
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const int i = wave + NW * j, r = 8 * i + (lane >> 3);
    const int row = j < 2 ? min(r, rows - 1) : r - BM;
    at[j] = row * pitch + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
  }
  LdsByte* const base = (LdsByte*)lds;
  auto request = [&](int chunk, int slot) __attribute__((always_inline)) {
    const int k = min(chunk, n_chunks - 1) * kRow;
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const int i = wave + NW * j;
      load_lds(j < 2 ? xs : ws, base + (slot * CH + 1024 * i), at[j], k);
    }
  };
#pragma unroll
  for (int c = 0; c < kDepth - 2; ++c) request(c, c);

  // this lane's piece of its row for each 16 numbers of a chunk; the same exchange for x and w
  const unsigned lds0 = (unsigned)(size_t)base;
  unsigned from[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) from[s] = lds0 + li * kRow + (((2 * s + lh) ^ ((li >> 1) & 7)) << 4);
  const unsigned x_at = 32 * kRow * rt, w_at = (BM + 32 * ct) * kRow;

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  auto mfma = [&](const u32x4& w, const u32x4& x) __attribute__((always_inline)) {
    if constexpr (F16)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, x), acc, 0, 0, 0);
    else
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
  };

  auto compute = [&](int slot) __attribute__((always_inline)) {
    const unsigned xb = slot * CH + x_at, wb = slot * CH + w_at;
    u32x4 x[4], w[4];
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %9\n\t"
        "ds_read_b128 %2, %10\n\t"
        "ds_read_b128 %3, %11\n\t"
        "ds_read_b128 %4, %12\n\t"
        "ds_read_b128 %5, %13\n\t"
        "ds_read_b128 %6, %14\n\t"
        "ds_read_b128 %7, %15\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(w[0]), "=&v"(x[0]), "=&v"(w[1]), "=&v"(x[1]), "=&v"(w[2]), "=&v"(x[2]), "=&v"(w[3]), "=&v"(x[3])
        : "v"(from[0] + wb), "v"(from[0] + xb), "v"(from[1] + wb), "v"(from[1] + xb), "v"(from[2] + wb),
          "v"(from[2] + xb), "v"(from[3] + wb), "v"(from[3] + xb)
        : "memory");
#pragma unroll
    for (int s = 0; s < 4; ++s) mfma(w[s], x[s]);
  };
  int slot = 0;
  for (int c = 0; c < n_chunks; c += 2) {
    constexpr int V = (kDepth - 4) * L;
    __builtin_amdgcn_s_waitcnt(0x0F70 | (V & 15) | (V >> 4) << 14);  // this wave's parts of chunks c, c + 1 are there
    __builtin_amdgcn_s_barrier();  // ... and the others'; chunks c - 2, c - 1 have been read
    __builtin_amdgcn_sched_barrier(0);
    const int before = slot == 0 ? kDepth - 2 : slot - 2;
    request(c + kDepth - 2, before);  // (past the end: the last one again, for no use)
    request(c + kDepth - 1, before + 1);
    __builtin_amdgcn_sched_barrier(0);
    compute(slot);
    if (c + 1 < n_chunks) compute(slot + 1);
    slot = slot + 2 == kDepth ? 0 : slot + 2;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // (nothing writes to LDS behind this workgroup's end)

  // D[i][j]: unit i = v % 4 + 4 * lh + 8 * (v / 4), row j = li
  const int m = m0 + 32 * rt + li;
  if (m >= g.M) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 r;
#pragma unroll
    for (int t = 0; t < 4; ++t) r[t] = fmaxf(acc[4 * q + t] + bias[q][t], 0.0f);
    const size_t o = (size_t)m * g.N + n0 + 32 * ct + 8 * q + 4 * lh;
    if constexpr (OUT_BF16) {
      u32x2 v;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const f32x2 pair = {r[2 * p], r[2 * p + 1]};
        v[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(pair, bf16x2));
      }
      *(u32x2*)((uint16_t*)g.out + o) = v;
    } else {
      *(f32x4*)((float*)g.out + o) = r;
    }
  }
}

template <int BM, bool F16, bool OUT_BF16>
hipError_t launch_t(const Fc16Args& g, hipStream_t st) {
  auto kern = fc16_kernel<BM, F16, OUT_BF16>;
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&] {
    attr_status = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
  });
  if (attr_status != hipSuccess) return attr_status;
  const int n_tiles = (g.M + BM - 1) / BM * (g.N / kBN);
  kern<<<(unsigned)((n_tiles + 7) / 8 * 8), 4 * BM, depth<BM>() * chunk_bytes<BM>(), st>>>(g);
  return hipGetLastError();
}
template <bool F16, bool OUT_BF16>
hipError_t launch_rows(const Fc16Args& g, hipStream_t st) {
  // the smallest tile whose grid is one round of workgroups
  const long long n_ct = g.N / kBN;
  if ((g.M + 31) / 32 * n_ct <= 256) return launch_t<32, F16, OUT_BF16>(g, st);
  if ((g.M + 63) / 64 * n_ct <= 256) return launch_t<64, F16, OUT_BF16>(g, st);
  return launch_t<128, F16, OUT_BF16>(g, st);
}

}  // namespace

// K in whole chunks (and rows that 32-bit offsets reach), N in whole tiles.
bool fc16_supported(int K, int N) { return K > 0 && K % 64 == 0 && K < (1 << 22) && N > 0 && N % kBN == 0; }

// x [M][K] and w [N][K] bf16 (or both fp16), 16-byte aligned; out fp32 or (out_bf16) bf16.
hipError_t launch_fc16(const void* x, const uint16_t* w, const float* bias, void* out, int M, int K, int N, int f16,
                       int out_bf16, hipStream_t st) {
  if (M == 0) return hipSuccess;
  if (!fc16_supported(K, N)) return hipErrorInvalidValue;
  const Fc16Args g{(const uint8_t*)x, (const uint8_t*)w, bias, out, M, N, K};
  if (f16) return out_bf16 ? launch_rows<true, true>(g, st) : launch_rows<true, false>(g, st);
  return out_bf16 ? launch_rows<false, true>(g, st) : launch_rows<false, false>(g, st);
}

}  // namespace sf
