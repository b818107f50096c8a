// Learner-side loss on a batch of trajectories (paper, Sec. 3.4: V-trace targets combined
// with PPO clipping; hyperparameter table of App. "VizDoom experiments"), forward values and
// the gradients with respect to the logits and the values.
//
//   ratio   = exp(logp_pi - logp_mu),  rho = min(rho_bar, ratio),  c = min(c_bar, ratio)
//   g_t     = gamma * (1 - done_t),    delta_t = rho_t * (r_t + g_t V_{t+1} - V_t)
//   vs_t - V_t = delta_t + g_t c_t (vs_{t+1} - V_{t+1}),   vs_T = V_T          (V-trace)
//   adv_t   = r_t + g_t vs_{t+1} - V_t
//   L_pi = -mean min(ratio adv, clamp(ratio, 1/clip, clip) adv),  L_v = c_v mean (V - vs)^2,
//   L_ent = -c_H mean entropy
//
// A sample's logits are reduced to the joint log-probability and the entropy; the backward recursion
// over time runs across the 32 or 64 lanes of a trajectory (the coefficient pairs are broadcast one
// by one, last step first); longer trajectories are walked in chunks from the end, carrying the
// recursion's value.  Targets, advantages, gradients and a workgroup's partial sums follow.  The
// partial sums are added in a fixed order, so the result does not depend on scheduling: by the
// workgroup that finds them all there (see publish), or by a second, single-workgroup launch.
//
// Memory side: the arrays are time-major, so the samples of a trajectory lie N * sumA floats apart
// and per-lane reads of a sample's logits touch a cache line per lane and element.  A workgroup
// therefore copies its trajectories' logits (and actions; one contiguous run of memory per time
// step) into LDS with coalesced loads (row pitch odd: walks over a sample's logits are free of bank
// conflicts), and the gradients leave for memory as contiguous runs again.  Tiles that do not fit
// LDS take the direct kernel (one wave per trajectory, one lane per time step).
#include <math.h>
#include <sys/random.h>
#include <time.h>

#include <atomic>
#include <mutex>

#include "sf_internal.h"

namespace sf {

namespace {

constexpr int kWave = 64;
constexpr int kTrajPerBlock = 4;

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, kWave);
  return v;
}

struct LossArgs {
  const float* logits;    // [T][N][sumA]
  const int32_t* actions; // [T][N][n_heads]
  const float* logp_mu;   // [T][N]
  const float* values;    // [T+1][N]
  const float* rewards;   // [T][N]
  const uint8_t* dones;   // [T][N]
  float* vs;              // [T][N]
  float* adv;             // [T][N]
  float* dlogits;         // [T][N][sumA] or null
  float* dvalues;         // [T][N] or null
  float* partials;        // [workgroups of the trajectory kernel][4], at most [N][4]; 16-byte aligned
  float* loss;            // [4]
  uint32_t key;           // of the partial sums' check words; 0: a second launch adds them
  int T, N, n_heads, sumA;
  int head_sizes[SF_MAX_HEADS];
  int head_off[SF_MAX_HEADS];    // first logit of each head
  int head_order[SF_MAX_HEADS];  // heads by size, largest first
  float gamma, rho_bar, c_bar, clip, critic_coef, entropy_coef;
};

__global__ __launch_bounds__(kWave* kTrajPerBlock) void appo_traj_kernel(LossArgs g) {
  const int lane = threadIdx.x % kWave;
  const int n = blockIdx.x * kTrajPerBlock + threadIdx.x / kWave;
  if (n >= g.N) return;  // whole wave leaves together; no block-level barrier below
  const float inv_m = 1.0f / ((float)g.T * (float)g.N);
  const float lo = 1.0f / g.clip, hi = g.clip;
  float sum_pi = 0.0f, sum_v = 0.0f, sum_ent = 0.0f;
  float carry = 0.0f;  // vs - V at the first step of the chunk after this one (0 at t = T)
  const int n_chunks = (g.T + kWave - 1) / kWave;
  for (int ch = n_chunks - 1; ch >= 0; --ch) {
    const int t = ch * kWave + lane;
    const bool live = t < g.T;
    const size_t s = (size_t)(live ? t : g.T - 1) * g.N + n;  // idle lanes re-read the last step
    // joint log-probability of the taken action and entropy, head by head
    float logp = 0.0f, ent = 0.0f;
    {
      const float* l = g.logits + s * g.sumA;
      for (int k = 0; k < g.n_heads; ++k) {
        const int A = g.head_sizes[k];
        float mx = -INFINITY;
        for (int i = 0; i < A; ++i) mx = fmaxf(mx, l[i]);
        float se = 0.0f;
        for (int i = 0; i < A; ++i) se += expf(l[i] - mx);
        const float lse = mx + logf(se);
        float hk = 0.0f;
        for (int i = 0; i < A; ++i) {
          const float ls = l[i] - lse;
          hk -= expf(ls) * ls;
        }
        const int a = min(max(g.actions[s * g.n_heads + k], 0), A - 1);
        logp += l[a] - lse;
        ent += hk;
        l += A;
      }
    }
    const float v = g.values[s], vn = g.values[s + g.N], r = g.rewards[s];
    const float gm = g.dones[s] ? 0.0f : g.gamma;
    const float ratio = expf(logp - g.logp_mu[s]);
    const float rho = fminf(g.rho_bar, ratio), c = fminf(g.c_bar, ratio);
    // idle lanes (past the last step) sit at the start of the backward scan: they pass 0 on
    const float delta = live ? rho * (r + gm * vn - v) : 0.0f;
    const float gc = live ? gm * c : 0.0f;
    float x = carry, mine = 0.0f;
    for (int l = kWave - 1; l >= 0; --l) {
      x = __shfl(delta, l, kWave) + __shfl(gc, l, kWave) * x;
      if (lane == l) mine = x;
    }
    // vs_{t+1} - V_{t+1}: the next lane's value, or the later chunk's first one
    float next = __shfl_down(mine, 1, kWave);
    if (lane == kWave - 1) next = carry;
    carry = __shfl(mine, 0, kWave);
    if (live) {
      const float vs = v + mine;
      const float adv = r + gm * (vn + next) - v;
      g.vs[s] = vs;
      g.adv[s] = adv;
      const float rc = fminf(fmaxf(ratio, lo), hi);
      const float a = ratio * adv, b = rc * adv;
      sum_pi -= fminf(a, b);
      const float dv = v - vs;
      sum_v += dv * dv;
      sum_ent -= ent;
      if (g.dvalues) g.dvalues[s] = 2.0f * g.critic_coef * dv * inv_m;
      if (g.dlogits) {
        const float dlp = a <= b ? -adv * ratio * inv_m : 0.0f;  // d L_pi / d logp_pi
        const float ce = g.entropy_coef * inv_m;
        const float* l = g.logits + s * g.sumA;
        float* d = g.dlogits + s * g.sumA;
        for (int k = 0; k < g.n_heads; ++k) {
          const int A = g.head_sizes[k];
          float mx = -INFINITY;
          for (int i = 0; i < A; ++i) mx = fmaxf(mx, l[i]);
          float se = 0.0f;
          for (int i = 0; i < A; ++i) se += expf(l[i] - mx);
          const float lse = mx + logf(se);
          float hk = 0.0f;
          for (int i = 0; i < A; ++i) {
            const float ls = l[i] - lse;
            hk -= expf(ls) * ls;
          }
          const int act = min(max(g.actions[s * g.n_heads + k], 0), A - 1);
          for (int i = 0; i < A; ++i) {
            const float ls = l[i] - lse;
            const float p = expf(ls);
            d[i] = dlp * ((i == act ? 1.0f : 0.0f) - p) + ce * p * (ls + hk);
          }
          l += A;
          d += A;
        }
      }
    }
  }
  sum_pi = wave_sum(sum_pi);
  sum_v = wave_sum(sum_v);
  sum_ent = wave_sum(sum_ent);
  if (lane == 0) {
    float* o = g.partials + (size_t)n * 4;
    o[0] = sum_pi;
    o[1] = sum_v;
    o[2] = sum_ent;
    o[3] = 0.0f;
  }
}

// floor(e / d) for e < 2^20, 1 <= d < 2^12, through the multiplier m = ceil(2^32 / d) (exact in
// that range: the excess e * (m * d - 2^32) stays below 2^32); d = 1 has no 32-bit multiplier.
__host__ __device__ inline uint32_t magic_of(uint32_t d) {
  return d <= 1 ? 0u : (uint32_t)((0x100000000ull + d - 1) / d);
}
__device__ inline uint32_t div_magic(uint32_t e, uint32_t d, uint32_t m) { return d <= 1 ? e : __umulhi(e, m); }

struct LdsPlan {
  int pitch;             // floats per sample row of the logits tile (odd, >= sumA)
  uint32_t m_sumA, m_nh; // multipliers for division by sumA and by n_heads,
  uint32_t m_row, m_row4, m_arow;  // by the length of a whole tile row (floats, 16-byte pieces; actions)
  int vec4;              // logits rows may be copied as 16-byte pieces (pitch == sumA, alignment)
};

constexpr int kLossThreads = kWave * kTrajPerBlock;

// Tile copies into LDS.  Row tt of the chunk holds, for time step t0 + tt, the nb trajectories'
// values side by side: memory run of nb * per elements at ((t0 + tt) * N + n0) * per, LDS sample
// (tt, j) at (tt * TPB + j) * pitch.  Loads are issued in batches of kCopyBatch per thread before
// the first of them is stored: a loop of load-then-store pays one memory latency per iteration.
constexpr int kCopyBatch = 8;

template <int TPB, int NT, typename T>
__device__ inline void copy_tile(const T* mem, T* tile, int t0, int nt, int N, int n0, int nb, int per,
                                 int pitch, uint32_t m_per, uint32_t m_row) {
  const int rowlen = nb * per;
  const int total = nt * rowlen;
  for (int e0 = threadIdx.x; e0 < total; e0 += NT * kCopyBatch) {
    T v[kCopyBatch];
    T* dst[kCopyBatch];
#pragma unroll
    for (int u = 0; u < kCopyBatch; ++u) {
      const int e = e0 + u * NT;
      const int ec = e < total ? e : total - 1;
      const int tt = (int)div_magic((uint32_t)ec, (uint32_t)rowlen, m_row);
      const int r = ec - tt * rowlen;
      const int j = (int)div_magic((uint32_t)r, (uint32_t)per, m_per);
      v[u] = mem[((size_t)(t0 + tt) * N + n0) * per + r];
      dst[u] = tile + (tt * TPB + j) * pitch + (r - j * per);
    }
#pragma unroll
    for (int u = 0; u < kCopyBatch; ++u)
      if (e0 + u * NT < total) *dst[u] = v[u];
  }
}

// The same for a full-width tile (nb == TPB) whose rows are contiguous in LDS as in memory
// (pitch == per) and 16-byte aligned on both sides: 16-byte pieces.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int TPB, int NT>
__device__ inline void copy_tile_vec4(const float* mem, float* tile, int t0, int nt, int N, int n0, int per,
                                      uint32_t m_row4) {
  const int row4 = TPB * per / 4;  // pieces per row
  const int total = nt * row4;
  for (int e0 = threadIdx.x; e0 < total; e0 += NT * kCopyBatch) {
    f32x4 v[kCopyBatch];
    f32x4* dst[kCopyBatch];
#pragma unroll
    for (int u = 0; u < kCopyBatch; ++u) {
      const int e = e0 + u * NT;
      const int ec = e < total ? e : total - 1;
      const int tt = (int)div_magic((uint32_t)ec, (uint32_t)row4, m_row4);
      const int r = ec - tt * row4;
      v[u] = *((const f32x4*)(mem + ((size_t)(t0 + tt) * N + n0) * per) + r);
      dst[u] = (f32x4*)(tile + (size_t)tt * TPB * per) + r;
    }
#pragma unroll
    for (int u = 0; u < kCopyBatch; ++u)
      if (e0 + u * NT < total) *dst[u] = v[u];
  }
}

// ---- adding the partial sums without a second launch ----
//
// A workgroup publishes its three sums with a check word (two 64-bit stores with device scope, past the
// caches that are not coherent across the XCDs; a store that has been waited for is seen by all) and then
// looks at the entries of all workgroups.  Stores and looks meet in memory in some order, so that the
// workgroup whose store came last finds all entries there.  The first to find them adds the sums in the
// fixed order, writes the losses and takes the entries back.  Nobody waits for another workgroup, and
// there is no counter: nothing of the caller's workspace has to be set ahead.  One wave does this while
// the others write the gradients: behind their stores it would wait for these.
//
// An entry that is taken back, or whose workgroup has begun, never passes for a published one: both its
// words differ from any published word, so half of it does not either.  A look may also find what was there before
// the call, where a workgroup has not begun.  Only its check word keeps that out: 31 bits, a function of the sums and
// of a key that each launch has for itself (replays of a recorded one share it), so that an entry of another call fits by chance only, and it is asked
// only as long as its workgroup has not begun while all others are done.  (The entry's number in it, too, cost
// 0.1 us of 16.8.)
//
// Whole calls, 41 logits in 7 heads, 32 steps (us, against the second launch, which is dependent on the
// first and costs 3.5 of the host's time, 13 us per call with it): 64 trajectories 12.3 -> 10.6, 256 12.3 -> 11.2,
// 512 13.1 -> 12.9, 700 13.4 -> 12.4, 1024 14.1 -> 13.4, 2048 17.4 -> 15.9, 4096 (512 workgroups) 23.7 -> 21.9.
typedef unsigned long long u64;
constexpr u64 kNoSums = ~0ull, kNoCheck = 0;
__device__ inline uint32_t check_word(uint32_t a, uint32_t b, uint32_t c, uint32_t key) {
  uint32_t h = a * 0x85EBCA6Bu + key;
  h = (h ^ (h >> 15) ^ b) * 0xC2B2AE35u;
  h = (h ^ (h >> 13) ^ c) * 0x9E3779B1u;
  return (h ^ (h >> 16)) | 1u;
}
__device__ inline void take_back(float* partials, int at) {
  u64* e = (u64*)partials + 2 * (size_t)at;
  __hip_atomic_store(e, kNoSums, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(e + 1, kNoCheck, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// by one lane; returns when the entry is in memory
__device__ inline void publish(float* partials, int at, const float (&sum)[3], uint32_t key) {
  uint32_t u[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) u[i] = sum[i] != sum[i] ? 0x7FC00000u : __builtin_bit_cast(uint32_t, sum[i]);
  u64* e = (u64*)partials + 2 * (size_t)at;
  __hip_atomic_store(e, u[0] | (u64)u[1] << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(e + 1, u[2] | (u64)check_word(u[0], u[1], u[2], key) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The order of the sums: 256 threads (i: entries i, i + 256, ...), then a binary tree over them.
constexpr int kReduceThreads = 256;
__device__ inline void write_losses(float pi, float v, float ent, float inv_m, float critic_coef, float entropy_coef,
                                    float* loss) {
  const float l_pi = pi * inv_m, l_v = critic_coef * v * inv_m, l_h = entropy_coef * ent * inv_m;
  loss[0] = l_pi;
  loss[1] = l_v;
  loss[2] = l_h;
  loss[3] = l_pi + l_v + l_h;
}

// The look of one wave at the n <= 256 * kLooks entries; lane l stands for threads l, l + 64, l + 128, l + 192.
// Many workgroups find all entries (they end at about the same time): the first of them, by an exchange,
// goes on (all of them taking all entries back made the call 3 to 10 us longer).  With more than kFew
// workgroups a look at sixteen neighbours comes first, since looks queue for the entries' few lines of
// memory: 512 workgroups 12.9 us per call against 14.8, 256 workgroups 11.5 against 11.2.
constexpr int kLooks = 2, kNear = 16, kFew = 256;
__device__ inline void entry(const LossArgs& g, int at, u64 (&w)[2]) {
  const u64* e = (const u64*)g.partials + 2 * (size_t)at;
#pragma unroll
  for (int q = 0; q < 2; ++q) w[q] = __hip_atomic_load(e + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool is_published(const LossArgs& g, const u64 (&w)[2]) {
  return w[0] != kNoSums && w[1] != kNoCheck &&
         (uint32_t)(w[1] >> 32) == check_word((uint32_t)w[0], (uint32_t)(w[0] >> 32), (uint32_t)w[1], g.key);
}
__device__ inline void add_if_complete(const LossArgs& g, int n, float inv_m) {
  const int lane = threadIdx.x & (kWave - 1);
  if (n > kFew) {
    u64 near[2];
    entry(g, min((int)blockIdx.x / kNear * kNear + lane % kNear, n - 1), near);
    if (!__all(is_published(g, near))) return;
  }
  u64 w[kLooks][4][2];
#pragma unroll
  for (int i = 0; i < kLooks; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) entry(g, min(kReduceThreads * i + kWave * k + lane, n - 1), w[i][k]);
  float sum[4][3] = {};
  bool there = true;
#pragma unroll
  for (int i = 0; i < kLooks; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      there = there && is_published(g, w[i][k]);
      if (kReduceThreads * i + kWave * k + lane < n) {
        sum[k][0] += __builtin_bit_cast(float, (uint32_t)w[i][k][0]);
        sum[k][1] += __builtin_bit_cast(float, (uint32_t)(w[i][k][0] >> 32));
        sum[k][2] += __builtin_bit_cast(float, (uint32_t)w[i][k][1]);
      }
    }
  if (!__all(there)) return;
  // the first of those who find all entries: it takes the first check word
  u64 first = 0;
  if (lane == 0) first = __hip_atomic_exchange((u64*)g.partials + 1, kNoCheck, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (!__any(first != kNoCheck)) return;
  float all[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    float a = (sum[0][q] + sum[2][q]) + (sum[1][q] + sum[3][q]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) a += __shfl_down(a, m, kWave);
    all[q] = a;
  }
  if (lane == 0) write_losses(all[0], all[1], all[2], inv_m, g.critic_coef, g.entropy_coef, g.loss);
  for (int i = lane; i < n; i += kWave) take_back(g.partials, i);
}

// A workgroup of NT threads owns TPB trajectories, LW (32 when T <= 32, else 64) time steps of them
// at a time.  What bounds it is the latency of a few dependent stretches, so each of them is spread
// over all threads:
//   1. tiles of logits and actions into LDS, coalesced;
//   2. one thread per (sample, head), largest heads first: log-sum-exp, entropy, log-probability;
//   3. one thread per sample: ratio, the backward recursion across the lanes of a trajectory,
//      targets, advantages, partial sums;
//   4. one thread per logit (four neighbouring ones where the rows allow): gradients straight from
//      the tile to memory; the partial sums meanwhile by the first wave (publish, add_if_complete).
// (One lane per sample through all of it, two waves per workgroup, took 14.5 us at 64 trajectories of
// 32 steps and seven heads, 19.6 at 2048; now 9.4 and 15.7, 1.6 TB/s of logits, actions and gradients:
// see pick_tile for whole calls.  The argument's three arrays of 16 and the addresses do not fit the scalar registers: 103 to 118
// of them are spilled to lanes with 32 lanes per trajectory, 41 to 55 with 64; what that costs has not been measured.)
// Per head one exponential per logit forward,
//   d_i = l_i - max, e_i = exp(d_i), se = sum e_i, sd = sum e_i d_i
//   lse = max + log se,  entropy = log se - sd / se   (= -sum p_i (l_i - lse))
// and one more for the gradient (p_i = exp(l_i - lse)).  These exponentials (arguments <= 0,
// results only ever summed or multiplied into terms of the 1e-4 tolerance) use the hardware
// exp2 (about 2 ulp for arguments of a few units); the logarithm per head and the importance
// ratio stay on the accurate routines.
template <int LW, int TPB, int NT>
__global__ __launch_bounds__(NT) void appo_traj_lds_kernel(LossArgs g, LdsPlan plan) {
  constexpr int S = LW * TPB;  // samples per chunk; sample (tt, j) of the tile is tt * TPB + j
  static_assert(S <= NT, "one thread per sample");
  extern __shared__ __attribute__((aligned(16))) float lds_tile[];
  const int hp = g.n_heads | 1;                              // odd pitch of the per-head values
  float* ltile = lds_tile;                                   // [S][pitch] logits
  float* t_lse = ltile + S * plan.pitch;                     // [S][hp]
  float* t_ent = t_lse + S * hp;                             // [S][hp]
  float* t_lp = t_ent + S * hp;                              // [S][hp] log-probability of the action taken
  int32_t* t_act = (int32_t*)(t_lp + S * hp);                // [S][hp] actions, then their place among the logits
  float* t_dlp = (float*)(t_act + S * hp);                   // [S] d L_pi / d logp_pi
  float* t_sum = t_dlp + S;                                  // [TPB][4] partial sums
  int32_t* head_of = (int32_t*)(t_sum + TPB * 4);            // [sumA] head of a logit
  // time step, trajectory of a sample (threads from S on ask for the same scalars again)
  const int tid = threadIdx.x, lane = tid % LW, j = tid / LW % TPB;
  const int n0 = blockIdx.x * TPB;
  const int nb = g.N - n0 < TPB ? g.N - n0 : TPB;
  const int n = n0 + j;
  const bool have = tid < S && n < g.N;
  const bool vec4 = plan.vec4 && nb == TPB;
  uint32_t m_row = plan.m_row, m_arow = plan.m_arow;
  if (nb != TPB) {
    m_row = magic_of((uint32_t)(nb * g.sumA));
    m_arow = magic_of((uint32_t)(nb * g.n_heads));
  }
  const float inv_m = 1.0f / ((float)g.T * (float)g.N);
  const float lo = 1.0f / g.clip, hi = g.clip;
  const float ce = g.entropy_coef * inv_m;
  // (the arguments' tables, read by a lane's own index, are a chain of memory latencies)
  __shared__ int t_size[SF_MAX_HEADS], t_off[SF_MAX_HEADS], t_order[SF_MAX_HEADS];
  if (tid < SF_MAX_HEADS) {
    t_size[tid] = g.head_sizes[tid];
    t_off[tid] = g.head_off[tid];
    t_order[tid] = g.head_order[tid];
  }
  float sum_pi = 0.0f, sum_v = 0.0f, sum_ent = 0.0f;
  float carry = 0.0f;
  if (g.key && tid == 0) take_back(g.partials, blockIdx.x);
  const int n_chunks = (g.T + LW - 1) / LW;
  for (int ch = n_chunks - 1; ch >= 0; --ch) {
    const int t0 = ch * LW;
    const int nt = g.T - t0 < LW ? g.T - t0 : LW;
    // the sample's scalars are requested first: their latency passes under the tile copies
    const int tt = t0 + lane < g.T ? lane : nt - 1;  // idle lanes re-read the chunk's last step
    const size_t s = (size_t)(t0 + tt) * g.N + (n < g.N ? n : g.N - 1);
    const float v = g.values[s], vn = g.values[s + g.N], r = g.rewards[s], lmu = g.logp_mu[s];
    const float gm = g.dones[s] ? 0.0f : g.gamma;
    if (vec4)
      copy_tile_vec4<TPB, NT>(g.logits, ltile, t0, nt, g.N, n0, g.sumA, plan.m_row4);
    else
      copy_tile<TPB, NT>(g.logits, ltile, t0, nt, g.N, n0, nb, g.sumA, plan.pitch, plan.m_sumA, m_row);
    copy_tile<TPB, NT>(g.actions, t_act, t0, nt, g.N, n0, nb, g.n_heads, hp, plan.m_nh, m_arow);
    __syncthreads();
    if (ch == n_chunks - 1)
      for (int i = tid; i < g.sumA; i += NT) {
        int k = 0;
        for (int q = 1; q < g.n_heads; ++q) k += i >= t_off[q];
        head_of[i] = k;
      }
    for (int w = tid; w < g.n_heads * S; w += NT) {
      const int k = t_order[w / S], smp = w % S;
      if (smp / TPB >= nt || smp % TPB >= nb) continue;
      const int A = t_size[k], off = t_off[k];
      const float* l = ltile + smp * plan.pitch + off;
      // four independent chains per pass: nobody else hides the latency of an LDS read or of an
      // exponential
      float m4[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      int i = 0;
      for (; i + 4 <= A; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) m4[u] = fmaxf(m4[u], l[i + u]);
      }
      for (; i < A; ++i) m4[0] = fmaxf(m4[0], l[i]);
      const float mx = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
      float se4[4] = {0.0f, 0.0f, 0.0f, 0.0f}, sd4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      for (i = 0; i + 4 <= A; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float d = l[i + u] - mx;
          const float e = __expf(d);
          se4[u] += e;
          sd4[u] = fmaf(e, d, sd4[u]);
        }
      }
      for (; i < A; ++i) {
        const float d = l[i] - mx;
        const float e = __expf(d);
        se4[0] += e;
        sd4[0] = fmaf(e, d, sd4[0]);
      }
      const float se = (se4[0] + se4[1]) + (se4[2] + se4[3]);
      const float sd = (sd4[0] + sd4[1]) + (sd4[2] + sd4[3]);
      const float lg = logf(se);
      const float lse = mx + lg;
      const int at = smp * hp + k;
      const int a = min(max(t_act[at], 0), A - 1);
      t_lse[at] = lse;
      t_ent[at] = lg - sd / se;
      t_lp[at] = l[a] - lse;
      t_act[at] = off + a;
    }
    __syncthreads();
    if (have) {
      const bool live = t0 + lane < g.T;
      const int smp = tt * TPB + j;
      float logp = 0.0f, ent = 0.0f;
      for (int k = 0; k < g.n_heads; ++k) {
        logp += t_lp[smp * hp + k];
        ent += t_ent[smp * hp + k];
      }
      const float ratio = expf(logp - lmu);
      const float rho = fminf(g.rho_bar, ratio), c = fminf(g.c_bar, ratio);
      const float delta = live ? rho * (r + gm * vn - v) : 0.0f;
      const float gc = live ? gm * c : 0.0f;
      float x = carry, mine = 0.0f;
      for (int l = LW - 1; l >= 0; --l) {
        x = __shfl(delta, l, LW) + __shfl(gc, l, LW) * x;
        if (lane == l) mine = x;
      }
      float next = __shfl_down(mine, 1, LW);
      if (lane == LW - 1) next = carry;
      carry = __shfl(mine, 0, LW);
      if (live) {
        const float vs = v + mine;
        const float adv = r + gm * (vn + next) - v;
        g.vs[s] = vs;
        g.adv[s] = adv;
        const float rc = fminf(fmaxf(ratio, lo), hi);
        const float a = ratio * adv, b = rc * adv;
        sum_pi -= fminf(a, b);
        const float dv = v - vs;
        sum_v += dv * dv;
        sum_ent -= ent;
        if (g.dvalues) g.dvalues[s] = 2.0f * g.critic_coef * dv * inv_m;
        t_dlp[smp] = a <= b ? -adv * ratio * inv_m : 0.0f;
      }
      if (ch == 0) {
#pragma unroll
        for (int m = LW / 2; m >= 1; m >>= 1) {
          sum_pi += __shfl_xor(sum_pi, m, LW);
          sum_v += __shfl_xor(sum_v, m, LW);
          sum_ent += __shfl_xor(sum_ent, m, LW);
        }
        if (lane == 0) {
          t_sum[j * 4] = sum_pi;
          t_sum[j * 4 + 1] = sum_v;
          t_sum[j * 4 + 2] = sum_ent;
        }
      }
    }
    __syncthreads();
    // one entry per workgroup, trajectories in order
    const bool adds = ch == 0 && g.key != 0;
    if (ch == 0 && (adds ? tid < kWave : tid == 0)) {
      if (tid == 0) {
        float sum[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          sum[i] = 0.0f;
          for (int q = 0; q < nb; ++q) sum[i] += t_sum[q * 4 + i];
        }
        if (adds)
          publish(g.partials, blockIdx.x, sum, g.key);
        else
          *(f32x4*)(g.partials + (size_t)blockIdx.x * 4) = f32x4{sum[0], sum[1], sum[2], 0.0f};
      }
      if (adds) add_if_complete(g, (int)gridDim.x, inv_m);
    }
    const int gt0 = adds ? tid - kWave : tid, gnt = adds ? NT - kWave : NT;  // threads of the gradients
    if (g.dlogits && gt0 >= 0) {
      auto gradient = [&](int smp, int i) {
        const int k = head_of[i], at = smp * hp + k;
        const float ls = ltile[smp * plan.pitch + i] - t_lse[at];
        const float p = __expf(ls);
        return t_dlp[smp] * ((i == t_act[at] ? 1.0f : 0.0f) - p) + ce * p * (ls + t_ent[at]);
      };
      if (vec4) {
        const int row4 = TPB * g.sumA / 4;
        for (int e = gt0; e < nt * row4; e += gnt) {
          const int gt = (int)div_magic((uint32_t)e, (uint32_t)row4, plan.m_row4), q = e - gt * row4;
          int jj = (int)div_magic((uint32_t)(4 * q), (uint32_t)g.sumA, plan.m_sumA), i = 4 * q - jj * g.sumA;
          f32x4 d;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            d[u] = gradient(gt * TPB + jj, i);
            if (++i == g.sumA) {
              i = 0;
              ++jj;
            }
          }
          *((f32x4*)(g.dlogits + ((size_t)(t0 + gt) * g.N + n0) * g.sumA) + q) = d;
        }
      } else {
        const int row = nb * g.sumA;
        for (int e = gt0; e < nt * row; e += gnt) {
          const int gt = (int)div_magic((uint32_t)e, (uint32_t)row, m_row), q = e - gt * row;
          const int jj = (int)div_magic((uint32_t)q, (uint32_t)g.sumA, plan.m_sumA), i = q - jj * g.sumA;
          g.dlogits[((size_t)(t0 + gt) * g.N + n0) * g.sumA + q] = gradient(gt * TPB + jj, i);
        }
      }
    }
    if (ch) __syncthreads();  // the tiles are free for the next chunk
  }
}

// Adds the partial sums (one entry per workgroup of the first launch) in an order that depends on
// their number only: thread i takes entries i, i + 256, ... (independent 16-byte loads), then a
// fixed binary tree over the 256 threads' sums in LDS (add_if_complete's order).
__global__ __launch_bounds__(kReduceThreads) void appo_reduce_kernel(const float* __restrict__ partials, int N,
                                                                     float inv_m, float critic_coef,
                                                                     float entropy_coef, float* __restrict__ loss) {
  __shared__ float red[3][kReduceThreads];
  const int tid = threadIdx.x;
  float a = 0.0f, b = 0.0f, c = 0.0f;
  for (int n = tid; n < N; n += kReduceThreads) {
    const f32x4 p = *(const f32x4*)(partials + (size_t)n * 4);
    a += p[0];
    b += p[1];
    c += p[2];
  }
  red[0][tid] = a;
  red[1][tid] = b;
  red[2][tid] = c;
  __syncthreads();
  for (int m = kReduceThreads / 2; m >= 1; m >>= 1) {
    if (tid < m) {
      red[0][tid] += red[0][tid + m];
      red[1][tid] += red[1][tid + m];
      red[2][tid] += red[2][tid + m];
    }
    __syncthreads();
  }
  if (tid == 0) write_losses(red[0][0], red[1][0], red[2][0], inv_m, critic_coef, entropy_coef, loss);
}

int check_loss_config(const sf_loss_config* c, const char* fn, int* sumA) {
  if (!c || c->struct_size != sizeof(sf_loss_config)) {
    set_error("%s: null configuration or struct_size mismatch", fn);
    return SF_ERR_ARG;
  }
  if (c->T < 1 || c->N < 1 || c->T > (1 << 20) || c->N > (1 << 24) || c->n_heads < 1 ||
      c->n_heads > SF_MAX_HEADS) {
    set_error("%s: T = %d, N = %d, n_heads = %d out of range", fn, c->T, c->N, c->n_heads);
    return SF_ERR_SHAPE;
  }
  int s = 0;
  for (int k = 0; k < c->n_heads; ++k) {
    if (c->head_sizes[k] < 1 || c->head_sizes[k] > 65535) {
      set_error("%s: head %d has size %d", fn, k, c->head_sizes[k]);
      return SF_ERR_SHAPE;
    }
    s += c->head_sizes[k];
  }
  if (!(c->clip >= 1.0f) || !(c->gamma >= 0.0f) || !(c->rho_bar > 0.0f) || !(c->c_bar > 0.0f)) {
    set_error("%s: clip must be >= 1, gamma >= 0, rho_bar and c_bar > 0", fn);
    return SF_ERR_SHAPE;
  }
  *sumA = s;
  return SF_OK;
}

}  // namespace
}  // namespace sf

using namespace sf;

extern "C" int64_t sf_appo_loss_workspace_bytes(const sf_loss_config* cfg) {
  int sumA;
  if (check_loss_config(cfg, "sf_appo_loss_workspace_bytes", &sumA) != SF_OK) return -1;
  // N x 4 partial sums, plus room to move a 4-byte aligned pointer up to a 16-byte boundary
  return (int64_t)cfg->N * 4 * (int64_t)sizeof(float) + 16;
}

namespace {

// The instantiations of the LDS-staged kernel: lanes per trajectory, trajectories per workgroup,
// threads.
struct LossTile {
  int lw, tpb, threads;
  void (*kernel)(LossArgs, LdsPlan);
};
template <int LW, int TPB, int NT>
constexpr LossTile loss_tile() { return LossTile{LW, TPB, NT, appo_traj_lds_kernel<LW, TPB, NT>}; }
const LossTile kTiles[] = {loss_tile<32, 8, 256>(), loss_tile<32, 4, 256>(), loss_tile<32, 8, 512>(),
                           loss_tile<32, 4, 512>(), loss_tile<32, 1, 256>(), loss_tile<64, 8, 512>(),
                           loss_tile<64, 4, 512>(), loss_tile<64, 2, 512>(), loss_tile<64, 1, 256>()};
constexpr size_t kMaxLds = 144 * 1024;

size_t tile_lds(const LossTile& k, int n_heads, int sumA) {
  const size_t pitch = sumA | 1, hp = n_heads | 1;
  return sizeof(float) * ((size_t)k.lw * k.tpb * (pitch + 4 * hp + 1) + k.tpb * 4 + sumA);
}

// Which of them takes a call: null if no chunk of a single trajectory fits LDS (the direct kernel
// does).  Several trajectories make the rows that a workgroup copies long runs of memory and its stages
// full, but too few workgroups leave CUs without one, and a large tile leaves a CU one workgroup.
// Whole calls, replayed from a graph (us; the kernel before had one lane per sample, 2 or 4
// waves):
//   logits x heads, steps x trajectories   before   1 of 256   4 of 256   4 of 512   8 of 256   8 of 512
//     7 x 1   32 x  700                       10.1       11.4        9.4        9.6       10.0        9.9
//     7 x 1   32 x 2048                       12.9       21.6       11.8       12.7       10.8       10.8
//     7 x 1   32 x 8192                       28.9       65.0       28.4       37.9       18.7       23.9
//    41 x 7   32 x   64                       15.8       11.0       14.1       12.5       18.9       15.2
//    41 x 7   32 x  700                       17.1       14.6       14.6       13.0       19.6       15.9
//    41 x 7   32 x 2048                       22.4       28.1       19.3       18.6       21.3       18.3
//    41 x 7   32 x 8192                       57.5       85.2       47.1       55.7       48.3       42.5
//    90 x 1   32 x 4096                       76.8       66.9       53.5       48.5       75.3       54.8
//    32 x 16  32 x 4096                       64.5       45.1       37.4       33.8       54.2       37.9
//    64 x 16  32 x  512                       34.0       13.6       22.5       16.8       35.9       24.6
//     7 x 1   64 x 4096                       30.0       49.0       26.4       31.9          -       23.0
//    15 x 1  128 x  600                       20.3       23.6       21.4       20.5          -       25.4
//    41 x 7   64 x 1024                       21.0       24.7       23.4       19.8          -       26.1
//    78 x 16  40 x 1024                       37.6       25.2   (four trajectories do not fit: 96 by the direct kernel)
// and 7 x 1, 64 x 300: 11.1, 11.4 one of 256, 10.7 two of 512.
const LossTile* pick_tile(int T, int N, int n_heads, int sumA) {
  const int lw = T <= 32 ? 32 : 64;
  const bool small = sumA <= 16, many = N >= 1536;
  int tpb, threads = 512;
  if (small) {
    tpb = many ? 8 : lw == 32 || N >= 512 ? 4 : 2;
    if (lw == 32) threads = 256;
  } else if (lw == 32) {
    tpb = many && sumA <= 48 ? 8 : N >= 640 ? 4 : 1;
  } else {
    tpb = N >= 1024 ? 4 : 1;
  }
  for (const LossTile& k : kTiles) {
    if (k.lw != lw || k.tpb > tpb || (k.tpb > 1 && k.threads != threads)) continue;
    if (tile_lds(k, n_heads, sumA) <= (k.tpb == 8 ? kMaxLds / 2 : kMaxLds)) return &k;
  }
  return nullptr;
}

// The check words' key of a launch with n entries, never zero: a number drawn once per process, and the launch's own.
const char g_key_tag = 0;  // (its address differs from process to process)
uint32_t launch_key(unsigned n) {
  static const uint32_t drawn = [] {
    uint32_t k = 0;
    if (getrandom(&k, sizeof(k), GRND_NONBLOCK) != (ssize_t)sizeof(k)) {
      timespec t{};
      (void)clock_gettime(CLOCK_REALTIME, &t);
      k = (uint32_t)t.tv_nsec * 0x9E3779B1u ^ (uint32_t)t.tv_sec ^ (uint32_t)((uintptr_t)&g_key_tag >> 12);
    }
    return k;
  }();
  static std::atomic<uint32_t> launches{0};
  const uint32_t k = drawn + launches.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B1u;
  return (k ^ n * 0x85EBCA6Bu) | 1u;
}

// Up to this many workgroups add the partial sums themselves (see add_if_complete; more take several
// rounds, where the second launch is the smaller part).
constexpr unsigned kOneLaunch = kLooks * kReduceThreads;

// Argument checks and the launches shared by the entry points; `partials` is 16-byte aligned device
// memory for N x 4 floats.
int run_appo_loss(const char* fn, const sf_loss_config* cfg, int sumA, const float* logits,
                  const int32_t* actions, const float* logp_mu, const float* values, const float* rewards,
                  const uint8_t* dones, float* vs, float* adv, float* loss, float* dlogits_opt,
                  float* dvalues_opt, float* partials, hipStream_t st) {
  if (!logits || !actions || !logp_mu || !values || !rewards || !dones || !vs || !adv || !loss ||
      !partials) {
    set_error("%s: null buffer", fn);
    return SF_ERR_ARG;
  }
  const void* al[] = {logits, actions, logp_mu, values, rewards, vs, adv, loss, dlogits_opt, dvalues_opt,
                      partials};
  for (const void* q : al)
    if ((reinterpret_cast<uintptr_t>(q) & 3) != 0) {
      set_error("%s: misaligned buffer (4 bytes)", fn);
      return SF_ERR_ARG;
    }
  LossArgs g;
  g.logits = logits; g.actions = actions; g.logp_mu = logp_mu; g.values = values; g.rewards = rewards;
  g.dones = dones; g.vs = vs; g.adv = adv; g.dlogits = dlogits_opt; g.dvalues = dvalues_opt;
  g.partials = partials; g.loss = loss; g.key = 0;
  g.T = cfg->T; g.N = cfg->N; g.n_heads = cfg->n_heads; g.sumA = sumA;
  for (int k = 0; k < SF_MAX_HEADS; ++k) g.head_sizes[k] = k < cfg->n_heads ? cfg->head_sizes[k] : 0;
  g.gamma = cfg->gamma; g.rho_bar = cfg->rho_bar; g.c_bar = cfg->c_bar; g.clip = cfg->clip;
  g.critic_coef = cfg->critic_coef; g.entropy_coef = cfg->entropy_coef;
  {
    int off = 0;
    for (int k = 0; k < SF_MAX_HEADS; ++k) {
      g.head_off[k] = off;
      off += g.head_sizes[k];
      g.head_order[k] = k;
    }
    for (int k = 1; k < g.n_heads; ++k)  // (a stable insertion sort: equal heads keep their order)
      for (int q = k; q > 0 && g.head_sizes[g.head_order[q]] > g.head_sizes[g.head_order[q - 1]]; --q) {
        const int o = g.head_order[q];
        g.head_order[q] = g.head_order[q - 1];
        g.head_order[q - 1] = o;
      }
  }
  const LossTile* tile = pick_tile(cfg->T, cfg->N, cfg->n_heads, sumA);
  const int TPB = tile ? tile->tpb : 1;
  LdsPlan plan;
  plan.pitch = sumA | 1;
  plan.m_sumA = magic_of((uint32_t)sumA);
  plan.m_nh = magic_of((uint32_t)cfg->n_heads);
  plan.m_row = magic_of((uint32_t)(TPB * sumA));
  plan.m_row4 = magic_of((uint32_t)(TPB * sumA / 4));
  plan.m_arow = magic_of((uint32_t)(TPB * cfg->n_heads));
  plan.vec4 = plan.pitch == sumA && (TPB * sumA) % 4 == 0 && ((size_t)cfg->N * sumA) % 4 == 0 &&
              ((uintptr_t)logits & 15) == 0 && (!dlogits_opt || ((uintptr_t)dlogits_opt & 15) == 0);
  static std::once_flag once;
  static hipError_t attr_status = hipSuccess;
  std::call_once(once, [&] {
    for (const LossTile& k : kTiles)
      if (attr_status == hipSuccess)
        attr_status = hipFuncSetAttribute((const void*)k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
  });
  if (attr_status != hipSuccess) {
    set_error("%s: hipFuncSetAttribute failed: %s", fn, hipGetErrorString(attr_status));
    return SF_ERR_DEVICE;
  }
  unsigned n_partials = (unsigned)((cfg->N + TPB - 1) / TPB);
  if (tile) {
    if (n_partials <= kOneLaunch) g.key = launch_key(n_partials);
    tile->kernel<<<n_partials, tile->threads, tile_lds(*tile, cfg->n_heads, sumA), st>>>(g, plan);
  } else {
    n_partials = (unsigned)cfg->N;
    appo_traj_kernel<<<(unsigned)((cfg->N + kTrajPerBlock - 1) / kTrajPerBlock), kLossThreads, 0, st>>>(g);
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && g.key == 0) {
    appo_reduce_kernel<<<1, kReduceThreads, 0, st>>>(g.partials, (int)n_partials, 1.0f / ((float)cfg->T * (float)cfg->N),
                                            cfg->critic_coef, cfg->entropy_coef, loss);
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    set_error("%s: launch failed: %s", fn, hipGetErrorString(e));
    return SF_ERR_DEVICE;
  }
  return SF_OK;
}

// Scratch of the entry point that allocates nothing: the partial sums.  One copy
// of this array exists on every GPU the library is loaded on, at an address of its own; host
// code never uses the symbol's name as an address but the pointer that hipGetSymbolAddress
// returns for the current device, looked up once per device.
constexpr int kStaticMaxTraj = 16384;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) float scratch[(size_t)kStaticMaxTraj * 4];
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(const char* fn, float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    set_error("%s: no current HIP device (%s)", fn, hipGetErrorString(e));
    return SF_ERR_DEVICE;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    float* ptr = nullptr;
    e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      set_error("%s: hipGetSymbolAddress failed on device %d: %s", fn, dev, hipGetErrorString(e));
      return SF_ERR_DEVICE;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return SF_OK;
}

}  // namespace

extern "C" int sf_appo_loss(const sf_loss_config* cfg, const float* logits, const int32_t* actions,
                            const float* logp_mu, const float* values, const float* rewards,
                            const uint8_t* dones, float* vs, float* adv, float* loss,
                            float* dlogits_opt, float* dvalues_opt, void* workspace, void* hip_stream) {
  static const char* fn = "sf_appo_loss";
  int sumA;
  int rc = check_loss_config(cfg, fn, &sumA);
  if (rc != SF_OK) return rc;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 3) != 0) {
    set_error("%s: null or misaligned workspace", fn);
    return SF_ERR_ARG;
  }
  return run_appo_loss(fn, cfg, sumA, logits, actions, logp_mu, values, rewards, dones, vs, adv, loss,
                       dlogits_opt, dvalues_opt,
                       reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(workspace) + 15) & ~(uintptr_t)15),
                       reinterpret_cast<hipStream_t>(hip_stream));
}

extern "C" int32_t sf_appo_loss_static_max_trajectories(void) { return kStaticMaxTraj; }

extern "C" int sf_appo_loss_static(const sf_loss_config* cfg, const float* logits, const int32_t* actions,
                                   const float* logp_mu, const float* values, const float* rewards,
                                   const uint8_t* dones, float* vs, float* adv, float* loss,
                                   float* dlogits_opt, float* dvalues_opt, void* hip_stream) {
  static const char* fn = "sf_appo_loss_static";
  int sumA;
  int rc = check_loss_config(cfg, fn, &sumA);
  if (rc != SF_OK) return rc;
  if (cfg->N > kStaticMaxTraj) {
    set_error("%s: N = %d trajectories exceed the built-in scratch (%d); use sf_appo_loss with a workspace",
              fn, cfg->N, kStaticMaxTraj);
    return SF_ERR_SHAPE;
  }
  float* partials = nullptr;
  rc = static_scratch(fn, &partials);
  if (rc != SF_OK) return rc;
  // nothing to clear: what an earlier call left is told apart from this one's (see publish, add_if_complete)
  return run_appo_loss(fn, cfg, sumA, logits, actions, logp_mu, values, rewards, dones, vs, adv, loss,
                       dlogits_opt, dvalues_opt, partials, reinterpret_cast<hipStream_t>(hip_stream));
}
