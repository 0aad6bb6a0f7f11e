// loss_kernels.h -- the streaming part of the path: importance ratio, clip, advantage weighting and the
// masked sequence / batch means (paper Sec. 6 display equation; App. A for the PPO mode).
// HBM-bound when large: ~21 bytes per token in, 4 out; two launches: per-generation lengths, then the tokens.  A batch
// one workgroup can hold takes one launch.  Reductions use wavefront cross-lane moves, then one fixed-order cross-block
// sum in fp64 (run by whichever block finishes last), so results are bitwise reproducible.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace llamarl {

constexpr int LOSS_ITEMS = 4;                                 // tokens per thread and step
constexpr int LOSS_MAX_BLOCKS = 512;                          // k_loss_tokens strides over the batch beyond this
constexpr int LOSS_NSUM = 5;                                  // loss, sum r, clipped count, sum delta, valid count

struct LossArgs {
  const float* logp;
  const float* mu_logp;
  const float* adv;
  const uint8_t* mask;
  const int32_t* targets;
  int64_t V;
  int64_t B, T;
  int adv_per_token;
  float rho;
  int clip_mode;
  float eps_lo, eps_hi;
  int norm_mode;
  int32_t* seq_len;    // [B] valid tokens per generation
  int32_t* seq_bad;    // [B] unmasked tokens with an out-of-range target
  double* partials;    // [nblocks][LOSS_NSUM]
  int nblocks;
  unsigned int* ticket;  // blocks of k_loss_tokens that have stored their partials (zeroed by k_seq_lengths)
  float* coef;
  float* loss;
  float* stats;
};

// Sum over the 64 lanes of a wavefront, the same value in every lane.  Rotations inside rows of 16 lanes (DPP), then the
// lane-group swaps: all on the VALU -- a shuffle tree goes through the LDS pipe twelve times per fp64 value, and the
// kernels below wait for five such values twice.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
constexpr int ROW_ROR(int n) { return 0x120 + n; }      // DPP control: rotate right by n inside a row
template <typename V, typename F>
__device__ __forceinline__ V move_words(V v, F f) {
  if constexpr (sizeof(V) == 8) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(V, ((uint64_t)f((uint32_t)(u >> 32)) << 32) | f((uint32_t)u));
  } else {
    return __builtin_bit_cast(V, f(__builtin_bit_cast(uint32_t, v)));
  }
}
template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
  v += move_words(v, [](uint32_t x) { return dpp_move<ROW_ROR(8)>(x); });
  v += move_words(v, [](uint32_t x) { return dpp_move<ROW_ROR(4)>(x); });
  v += move_words(v, [](uint32_t x) { return dpp_move<ROW_ROR(2)>(x); });
  v += move_words(v, [](uint32_t x) { return dpp_move<ROW_ROR(1)>(x); });
  // swapping a register with a copy of itself leaves the own value and the other half's, in either order
  v = move_words(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false)[0]; }) +
      move_words(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false)[1]; });
  v = move_words(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false)[0]; }) +
      move_words(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false)[1]; });
  return v;
}

// Four neighbouring tokens t0 .. t0+3 (t0 a multiple of 4) that one thread works on.  logp, mu_logp, targets, coef and a
// per-token advantage start 16-byte aligned, the mask 4-byte aligned: one load each, except for the last, partial
// group of the batch, which goes token by token.
struct TokenGroup {
  float lp[4], mu[4], ad[4];
  bool ok[4], bad[4];      // valid; unmasked, but the target is out of range

  __device__ __forceinline__ void load_flags(const LossArgs& a, int64_t t0, int64_t N) {
    uint8_t mk[4] = {1, 1, 1, 1};
    int tg[4] = {0, 0, 0, 0};
    if (t0 + 4 <= N) {
      if (a.mask != nullptr) {
        const uchar4 k = *reinterpret_cast<const uchar4*>(a.mask + t0);
        mk[0] = k.x; mk[1] = k.y; mk[2] = k.z; mk[3] = k.w;
      }
      if (a.targets != nullptr) {
        const int4 y = *reinterpret_cast<const int4*>(a.targets + t0);
        tg[0] = y.x; tg[1] = y.y; tg[2] = y.z; tg[3] = y.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (t0 + i >= N) {
          mk[i] = 0;
          continue;
        }
        if (a.mask != nullptr) mk[i] = a.mask[t0 + i];
        if (a.targets != nullptr) tg[i] = a.targets[t0 + i];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bad[i] = mk[i] != 0 && a.targets != nullptr && (tg[i] < 0 || (int64_t)tg[i] >= a.V);
      ok[i] = mk[i] != 0 && !bad[i];
    }
  }
  __device__ __forceinline__ void load_values(const LossArgs& a, int64_t t0, int64_t N) {
    if (t0 + 4 <= N) {
      const float4 l = *reinterpret_cast<const float4*>(a.logp + t0);
      const float4 m = *reinterpret_cast<const float4*>(a.mu_logp + t0);
      lp[0] = l.x; lp[1] = l.y; lp[2] = l.z; lp[3] = l.w;
      mu[0] = m.x; mu[1] = m.y; mu[2] = m.z; mu[3] = m.w;
      if (a.adv_per_token) {
        const float4 v = *reinterpret_cast<const float4*>(a.adv + t0);
        ad[0] = v.x; ad[1] = v.y; ad[2] = v.z; ad[3] = v.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t t = min(t0 + i, N - 1);
        lp[i] = a.logp[t];
        mu[i] = a.mu_logp[t];
        if (a.adv_per_token) ad[i] = a.adv[t];
      }
    }
  }
  // ratio, clip, weight: stores coef, adds the five sums.  len(b) = valid tokens of generation b.
  template <typename Len>
  __device__ __forceinline__ void finish(const LossArgs& a, int64_t t0, int64_t N, float n_valid, float b_valid, Len len,
                                         double (&acc)[LOSS_NSUM]) const {
    int64_t b, in_b;                              // generation of the first token; later ones step over the edge
    if (N <= 0xffffffffll) {
      const uint32_t q = (uint32_t)t0 / (uint32_t)a.T;
      b = q;
      in_b = (uint32_t)t0 - q * (uint32_t)a.T;
    } else {
      b = t0 / a.T;
      in_b = t0 - b * a.T;
    }
    float c4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      while (in_b >= a.T) {
        in_b -= a.T;
        ++b;
      }
      ++in_b;
      c4[i] = 0.f;
      if (!ok[i]) continue;
      const float delta = lp[i] - mu[i];
      const float r = expf(delta);
      const float A = a.adv_per_token ? ad[i] : a.adv[b];
      float Z;
      if (a.norm_mode == 0) Z = n_valid;
      else if (a.norm_mode == 1) Z = b_valid * (float)max(len(b), 1);
      else Z = (float)a.B;
      bool clipped;
      float term, c;
      if (a.clip_mode == 0) {
        const float w = fminf(r, a.rho);          // one-sided clip from above; w is a constant weight
        c = -(w * A) / Z;
        clipped = r > a.rho;
        term = c * lp[i];
      } else {
        const float rc = fminf(fmaxf(r, 1.f - a.eps_lo), 1.f + a.eps_hi);
        const float u = r * A, k = rc * A;
        const bool active = u <= k;               // the unclipped term is the min: gradient flows through r
        c = active ? -(A * r) / Z : 0.f;
        clipped = !active;
        term = -fminf(u, k) / Z;
      }
      c4[i] = c;
      acc[0] += (double)term;
      acc[1] += (double)r;
      acc[2] += clipped ? 1.0 : 0.0;
      acc[3] += (double)delta;
      acc[4] += 1.0;
    }
    if (t0 + 4 <= N) {
      *reinterpret_cast<float4*>(a.coef + t0) = make_float4(c4[0], c4[1], c4[2], c4[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (t0 + i < N) a.coef[t0 + i] = c4[i];
    }
  }
};

__device__ __forceinline__ void write_loss_stats(const LossArgs& a, const double (&t)[LOSS_NSUM], double bad) {
  const double den = t[4] > 0 ? t[4] : 1.0;
  a.loss[0] = (float)t[0];
  a.stats[0] = (float)t[4];
  a.stats[1] = (float)(t[1] / den);
  a.stats[2] = (float)(t[2] / den);
  a.stats[3] = (float)(t[3] / den);
  a.stats[4] = (float)bad;
}

// The whole loss of a small batch in one workgroup and one launch: flags and values of every token are loaded first,
// the per-generation counts meet in LDS, and no partial sum leaves the workgroup.  Bound by latency up to ~4 k tokens
// (launch, one trip to memory, three reductions) and by one CU's VALU beyond.  Against the two launches: 256 tokens
// 9.9 -> 5.0 us, 4096 11.0 -> 6.4, 8192 11.2 -> 8.7; at 16384 it is 11.8, no better than they are.
constexpr int LOSS_SMALL_THREADS = 1024;
constexpr int LOSS_SMALL_GROUPS = 2;
constexpr int64_t LOSS_SMALL_TOKENS = (int64_t)LOSS_SMALL_GROUPS * LOSS_SMALL_THREADS * LOSS_ITEMS;   // 8192
constexpr int64_t LOSS_SMALL_GENERATIONS = LOSS_SMALL_THREADS;
__global__ __launch_bounds__(LOSS_SMALL_THREADS) void k_loss_small(LossArgs a) {
  constexpr int WAVES = LOSS_SMALL_THREADS / 64;
  __shared__ int s_len[LOSS_SMALL_GENERATIONS];
  __shared__ int s_red[3][WAVES];
  __shared__ double s_sum[LOSS_NSUM][WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t N = a.B * a.T;
  s_len[tid] = 0;
  TokenGroup g[LOSS_SMALL_GROUPS];
#pragma unroll
  for (int q = 0; q < LOSS_SMALL_GROUPS; ++q) {
    const int64_t t0 = (int64_t)(q * LOSS_SMALL_THREADS + tid) * 4;
    if (t0 < N) {
      g[q].load_flags(a, t0, N);
      g[q].load_values(a, t0, N);
    }
  }
  __syncthreads();
  int nbad = 0;
#pragma unroll
  for (int q = 0; q < LOSS_SMALL_GROUPS; ++q) {
    const uint32_t t0 = (uint32_t)(q * LOSS_SMALL_THREADS + tid) * 4u, T = (uint32_t)a.T;
    const bool in = (int64_t)t0 < N;
    int cnt = 0;
    if (in) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        cnt += g[q].ok[i] ? 1 : 0;
        nbad += g[q].bad[i] ? 1 : 0;
      }
    }
    const uint32_t first = t0 - 4u * (uint32_t)lane;               // the wavefront's 256 tokens
    const uint32_t b0 = first / T;
    if ((int64_t)first < N && min((int64_t)first + 255, N - 1) < (int64_t)(b0 + 1) * T) {   // wave-uniform: one generation
      cnt = wave_sum(cnt);
      if (lane == 0 && cnt > 0) atomicAdd(&s_len[b0], cnt);
    } else if (in) {
      uint32_t b = t0 / T, in_b = t0 - b * T;
      cnt = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (in_b >= T) {
          if (cnt > 0) atomicAdd(&s_len[b], cnt);
          cnt = 0;
          in_b = 0;
          ++b;
        }
        ++in_b;
        cnt += g[q].ok[i] ? 1 : 0;
      }
      if (cnt > 0) atomicAdd(&s_len[b], cnt);
    }
  }
  __syncthreads();
  const int l = tid < (int)a.B ? s_len[tid] : 0;
  const int nv_w = wave_sum(l), bv_w = wave_sum(l > 0 ? 1 : 0), bad_w = wave_sum(nbad);
  if (lane == 0) {
    s_red[0][wave] = nv_w;
    s_red[1][wave] = bv_w;
    s_red[2][wave] = bad_w;
  }
  __syncthreads();
  int nv = 0, bv = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    nv += s_red[0][w];
    bv += s_red[1][w];
  }
  const float n_valid = (float)(nv > 0 ? nv : 1), b_valid = (float)(bv > 0 ? bv : 1);
  double acc[LOSS_NSUM] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < LOSS_SMALL_GROUPS; ++q) {
    const int64_t t0 = (int64_t)(q * LOSS_SMALL_THREADS + tid) * 4;
    if (t0 < N) g[q].finish(a, t0, N, n_valid, b_valid, [&](int64_t b) { return s_len[b]; }, acc);
  }
#pragma unroll
  for (int q = 0; q < LOSS_NSUM; ++q) {
    const double v = wave_sum(acc[q]);
    if (lane == 0) s_sum[q][wave] = v;
  }
  __syncthreads();
  if (tid == 0) {
    double t[LOSS_NSUM] = {0, 0, 0, 0, 0};
    int bad = 0;
    for (int w = 0; w < WAVES; ++w) {
#pragma unroll
      for (int q = 0; q < LOSS_NSUM; ++q) t[q] += s_sum[q][w];
      bad += s_red[2][w];
    }
    write_loss_stats(a, t, (double)bad);
  }
}

// One block per generation: valid-token count and bad-target count.  Groups of four tokens at multiples of four of the
// whole batch, so that every load is aligned whatever T is; the groups at the two ends are shared with the
// neighbouring generations.
// SEQ_THREADS: 1024 for long generations (few blocks, each with many groups in flight), 256 for short ones.
template <int SEQ_THREADS>
__global__ __launch_bounds__(SEQ_THREADS) void k_seq_lengths(LossArgs a) {
  const int64_t N = a.B * a.T, first = (int64_t)blockIdx.x * a.T, last = first + a.T;   // [first, last)
  int cnt = 0, nbad = 0;
#pragma unroll 4
  for (int64_t t0 = (first & ~(int64_t)3) + (int64_t)threadIdx.x * 4; t0 < last; t0 += SEQ_THREADS * 4) {
    TokenGroup g;
    g.load_flags(a, t0, N);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool mine = t0 + i >= first && t0 + i < last;
      cnt += mine && g.ok[i] ? 1 : 0;
      nbad += mine && g.bad[i] ? 1 : 0;
    }
  }
  cnt = wave_sum(cnt);
  nbad = wave_sum(nbad);
  __shared__ int s_c[SEQ_THREADS / 64], s_b[SEQ_THREADS / 64];
  if ((threadIdx.x & 63) == 0) {
    s_c[threadIdx.x >> 6] = cnt;
    s_b[threadIdx.x >> 6] = nbad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int c = 0, d = 0;
    for (int w = 0; w < SEQ_THREADS / 64; ++w) {
      c += s_c[w];
      d += s_b[w];
    }
    a.seq_len[blockIdx.x] = c;
    a.seq_bad[blockIdx.x] = d;
    if (blockIdx.x == 0) *a.ticket = 0u;
  }
}

// coef[t] and per-block partial sums; the block that finishes last adds the partials up in a fixed order (by
// block index, whichever block it is), so loss and statistics are bitwise reproducible without a third launch.
// HBM-bound on a large batch, where 512 blocks of 1024 threads fill the chip's wavefront slots; a batch those blocks
// would not cover takes blocks of 256 threads and more CUs instead.
template <int LOSS_THREADS>
__global__ __launch_bounds__(LOSS_THREADS, 8) void k_loss_tokens(LossArgs a) {
  constexpr int LOSS_BLOCK_TOKENS = LOSS_THREADS * LOSS_ITEMS;
  __shared__ long long s_red[2][LOSS_THREADS / 64];
  __shared__ double s_sum[LOSS_NSUM + 1][LOSS_THREADS / 64];
  __shared__ bool s_last;
  const int64_t N = a.B * a.T;
  // the first chunk's loads go out before the batch normaliser is known
  int64_t t0 = (int64_t)blockIdx.x * LOSS_BLOCK_TOKENS + (int64_t)threadIdx.x * LOSS_ITEMS;
  TokenGroup g;
  if (t0 < N) {
    g.load_flags(a, t0, N);
    g.load_values(a, t0, N);
  }
  // every block re-derives the batch normaliser from the B per-generation counts (B is small)
  long long nv = 0, bv = 0;
  for (int64_t b = threadIdx.x; b < a.B; b += LOSS_THREADS) {
    const int l = a.seq_len[b];
    nv += l;
    bv += (l > 0) ? 1 : 0;
  }
  nv = wave_sum(nv);
  bv = wave_sum(bv);
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = nv;
    s_red[1][threadIdx.x >> 6] = bv;
  }
  __syncthreads();
  nv = 0;
  bv = 0;
  for (int w = 0; w < LOSS_THREADS / 64; ++w) {
    nv += s_red[0][w];
    bv += s_red[1][w];
  }
  const float n_valid = (float)(nv > 0 ? nv : 1);
  const float b_valid = (float)(bv > 0 ? bv : 1);

  double acc[LOSS_NSUM] = {0, 0, 0, 0, 0};
  while (t0 < N) {
    const int64_t next = t0 + (int64_t)gridDim.x * LOSS_BLOCK_TOKENS;
    TokenGroup ng;
    if (next < N) {                               // the next chunk's loads fly under this chunk's arithmetic
      ng.load_flags(a, next, N);
      ng.load_values(a, next, N);
    }
    g.finish(a, t0, N, n_valid, b_valid, [&a](int64_t b) { return a.seq_len[b]; }, acc);
    g = ng;
    t0 = next;
  }
#pragma unroll
  for (int q = 0; q < LOSS_NSUM; ++q) {
    const double v = wave_sum(acc[q]);
    if ((threadIdx.x & 63) == 0) s_sum[q][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  // Publish the partials, then take a ticket: the block that draws the last one reads everybody's.  The partials are
  // device-scope atomic stores (they go past the XCD's private L2), complete when the wavefront's vmcnt is zero, and
  // are read back with device-scope atomic loads; the ticket follows that wait.  A __threadfence() would order more
  // than that -- it writes back every dirty line of the L2, coef among them, once per block.
  if (threadIdx.x < 64) {
    if (threadIdx.x < LOSS_NSUM) {
      double v = 0;
      for (int w = 0; w < LOSS_THREADS / 64; ++w) v += s_sum[threadIdx.x][w];
      __hip_atomic_store(a.partials + (int64_t)blockIdx.x * LOSS_NSUM + threadIdx.x, v, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0)
      s_last = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
               (unsigned int)a.nblocks - 1u;
  }
  __syncthreads();
  if (!s_last) return;                            // block-uniform

  double tot[LOSS_NSUM + 1] = {0, 0, 0, 0, 0, 0};
  for (int i = threadIdx.x; i < a.nblocks; i += LOSS_THREADS)
#pragma unroll
    for (int q = 0; q < LOSS_NSUM; ++q)           // device-scope loads: other CUs wrote these during this launch
      tot[q] += __hip_atomic_load(a.partials + (int64_t)i * LOSS_NSUM + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int64_t b = threadIdx.x; b < a.B; b += LOSS_THREADS) tot[LOSS_NSUM] += (double)a.seq_bad[b];
#pragma unroll
  for (int q = 0; q <= LOSS_NSUM; ++q) {
    const double v = wave_sum(tot[q]);
    if ((threadIdx.x & 63) == 0) s_sum[q][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t[LOSS_NSUM], bad = 0;
    for (int q = 0; q < LOSS_NSUM; ++q) {
      t[q] = 0;
      for (int w = 0; w < LOSS_THREADS / 64; ++w) t[q] += s_sum[q][w];
    }
    for (int w = 0; w < LOSS_THREADS / 64; ++w) bad += s_sum[LOSS_NSUM][w];
    write_loss_stats(a, t, bad);
  }
}

// One wavefront per prompt: mean (and optionally population std) of its n rewards by shuffles, fp64 accumulation.
__global__ __launch_bounds__(256) void k_group_advantages(const float* rewards, int64_t P, int64_t n, int normalise_std,
                                                          float eps, float* adv) {
  const int64_t p = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (p >= P) return;
  const float* r = rewards + p * n;
  double s = 0.0;
  for (int64_t i = lane; i < n; i += 64) s += (double)r[i];
  const double mean = wave_sum(s) / (double)n;
  double scale = 1.0;
  if (normalise_std) {
    double q = 0.0;
    for (int64_t i = lane; i < n; i += 64) {
      const double dlt = (double)r[i] - mean;
      q += dlt * dlt;
    }
    scale = 1.0 / (sqrt(wave_sum(q) / (double)n) + (double)eps);
  }
  for (int64_t i = lane; i < n; i += 64) adv[p * n + i] = (float)(((double)r[i] - mean) * scale);
}

// One block per generation: masked sum of the per-token log-ratios log pi - log pi_base (fp64, fixed order), then
// shaped = reward - lambda * sum.  Masking is a select, so NaN at masked positions never enters the sum.
// Bound by latency and by the loads one CU keeps in flight: groups of four tokens at multiples of four of the whole
// batch (16 + 16 + 4 bytes, aligned whatever T is; the end groups are shared with the neighbouring generations), 1024
// threads for long generations.  Unaligned arrays and the batch's last, partial group go token by token.  128
// generations of up to 16384 tokens: 36 us with 256 threads and one token per
// load, 5.5 us now; 2 generations 19 -> 4.4 us.
template <int KL_THREADS>
__global__ __launch_bounds__(KL_THREADS) void k_kl_shaped_rewards(const float* rewards, const float* logp,
                                                                  const float* base_logp, const uint8_t* mask, int64_t B,
                                                                  int64_t T, int aligned, float lambda_kl, float* shaped,
                                                                  float* kl) {
  __shared__ double s_w[KL_THREADS / 64];
  const int64_t b = blockIdx.x, N = B * T, first = b * T, last = first + T;
  double acc = 0.0;
#pragma unroll 4
  for (int64_t t0 = (first & ~(int64_t)3) + (int64_t)threadIdx.x * 4; t0 < last; t0 += KL_THREADS * 4) {
    float lp[4], bl[4];
    uint8_t mk[4] = {1, 1, 1, 1};
    if (aligned && t0 + 4 <= N) {
      const float4 l = *reinterpret_cast<const float4*>(logp + t0), r = *reinterpret_cast<const float4*>(base_logp + t0);
      lp[0] = l.x; lp[1] = l.y; lp[2] = l.z; lp[3] = l.w;
      bl[0] = r.x; bl[1] = r.y; bl[2] = r.z; bl[3] = r.w;
      if (mask != nullptr) {
        const uchar4 k = *reinterpret_cast<const uchar4*>(mask + t0);
        mk[0] = k.x; mk[1] = k.y; mk[2] = k.z; mk[3] = k.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t t = min(t0 + i, N - 1);
        lp[i] = logp[t];
        bl[i] = base_logp[t];
        if (mask != nullptr) mk[i] = mask[t];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool in = t0 + i >= first && t0 + i < last && mk[i] != 0;
      acc += in ? ((double)lp[i] - (double)bl[i]) : 0.0;
    }
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double k = 0.0;
    for (int w = 0; w < KL_THREADS / 64; ++w) k += s_w[w];
    if (kl != nullptr) kl[b] = (float)k;
    shaped[b] = (float)((double)rewards[b] - (double)lambda_kl * k);
  }
}

}  // namespace llamarl
