// The coin min(1, p(x) / q(x)) of one drafted token and, where it fails, the draw from the residual max(0, p - q): shared by the
// correction of rejected rows (k_control.hip) and the speculative-decoding windows (k_sd.hip).
#pragma once
#include <algorithm>
#include "dev.h"

namespace sprinter {

constexpr int COIN_THREADS = 256, COIN_U = 8, COIN_BLOCK = COIN_THREADS * COIN_U;   // words a workgroup holds in registers

// fold(v) over a workgroup of COIN_THREADS, in every thread.  s: one float of LDS per wave that nothing else uses.
template <bool MAX>
__device__ __forceinline__ float coin_fold(float v, float* s) {
  v = MAX ? wave_max(v) : wave_sum(v);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = s[0];
#pragma unroll
  for (int q = 1; q < COIN_THREADS / 64; ++q) r = MAX ? fmaxf(r, s[q]) : r + s[q];
  return r;
}

// Scratch of the tokens of one pass: what each slice of a token's vocabulary holds, the largest key, workgroups that gave theirs.
struct CoinWork { float4* part; u64* key; int* arrived; int S, blocks; };   // part [n][S]: maxima and sums (q, p) of a slice

// A block per workgroup up to 4096 workgroups (512: 80 tokens of 50257 words 40 us, 2048 and 4096: 28; 640 tokens 213 / 180 with
// 2048 / 4096), and as many slices as n tokens' partial results find room for in `bytes` (a scratch row has 4 bytes per QKV column).
constexpr int COIN_GRID = 4096;
inline CoinWork coin_work(void* work, size_t bytes, int n, int V) {
  const int all = (V + COIN_BLOCK - 1) / COIN_BLOCK;
  const long long room = ((long long)(bytes / n) - 12) / 16;
  const long long most = std::max(1LL, std::min<long long>(room, COIN_GRID / n));
  CoinWork w;
  w.blocks = (int)((all + most - 1) / most);
  w.S = (all + w.blocks - 1) / w.blocks;
  w.part = (float4*)work;
  w.key = (u64*)(w.part + (size_t)n * w.S);
  w.arrived = (int*)(w.key + n);
  return w;
}

// A maximum as the offset of exponents: where all words are -inf, so that their exponentials are 0 (and a NaN stays one).
__device__ __forceinline__ float coin_offset(float m) { return m == -INFINITY ? 0.f : m; }

struct CoinWords {                                       // logits / T of the words v0 + 256 u of a thread
  float q[COIN_U], p[COIN_U];
  __device__ __forceinline__ void load(const float* __restrict__ lq, const float* __restrict__ lp, int v0, int V, float it) {
#pragma unroll
    for (int u = 0; u < COIN_U; ++u) { const int v = min(v0 + u * COIN_THREADS, V - 1); q[u] = lq[v]; p[u] = lp[v]; }
#pragma unroll
    for (int u = 0; u < COIN_U; ++u) {                   // -inf beyond the vocabulary
      const bool in = v0 + u * COIN_THREADS < V;
      q[u] = in ? q[u] * it : -INFINITY;
      p[u] = in ? p[u] * it : -INFINITY;
    }
  }
};

// q = softmax(lq * it), p = softmax(lp * it); the coin fails with probability 1 - min(1, p(x) / q(x)), and only then a token is
// drawn from max(0, p - q): Gumbel-max on ln(p - q) with the noise of the target stream.  float32 throughout.
// Philox, two exponentials and two logarithms per word are the work (50257 words: most of 75 us on one compute unit), so a
// token's vocabulary is cut into w.S slices of w.blocks x 2048 words, a workgroup (blockIdx.y) each, in two launches: the maxima
// and sums of the slices; then every workgroup puts them together (in one order: the same coin everywhere) and draws from its
// slice, and the last one to arrive takes the largest key.  One slice needs one launch, and one block stays in registers.
// One workgroup of 16 waves per token, three sweeps over the rows -> this, us back to back: 1000 words, 1 / 80 tokens 10.0 -> 6.3,
// 10.5 -> 7.1; 32000 words, 4 tokens 48 -> 12.7; 50257 words, 4 / 24 / 80 / 640 tokens 75 -> 12.2, 75 -> 14.9, 77 -> 28, 242 -> 180;
// 128256 words, 24 tokens 176 -> 21.
// Grid: (tokens, S); i: the token's place in w.

// Maxima and sums of a slice, in every thread; x: its first block.
__device__ __forceinline__ float4 coin_sums(const float* __restrict__ lq, const float* __restrict__ lp, int V, float it, int first,
                                            int blocks, CoinWords& x) {
  __shared__ float s_fold[4][COIN_THREADS / 64];
  float mq = -INFINITY, mp = -INFINITY, sq = 0.f, sp = 0.f;
  for (int k = 0; k < blocks; ++k) {
    x.load(lq, lp, first + k * COIN_BLOCK, V, it);
#pragma unroll
    for (int u = 0; u < COIN_U; ++u) { mq = fmaxf(mq, x.q[u]); mp = fmaxf(mp, x.p[u]); }
  }
  mq = coin_fold<true>(mq, s_fold[0]);
  mp = coin_fold<true>(mp, s_fold[1]);
  const float oq = coin_offset(mq), op = coin_offset(mp);
  for (int k = blocks; k-- > 0;) {                       // (the last block is still there, and the first one stays)
    if (k != blocks - 1) x.load(lq, lp, first + k * COIN_BLOCK, V, it);
#pragma unroll
    for (int u = 0; u < COIN_U; ++u) { sq += expf(x.q[u] - oq); sp += expf(x.p[u] - op); }
  }
  return make_float4(mq, mp, coin_fold<false>(sq, s_fold[2]), coin_fold<false>(sp, s_fold[3]));
}

__device__ __forceinline__ void coin_slice(const float* __restrict__ lq, const float* __restrict__ lp, int V, float it,
                                           const CoinWork& w, int i) {
  const int tid = threadIdx.x, slice = blockIdx.y;
  CoinWords x;
  const float4 r = coin_sums(lq, lp, V, it, slice * w.blocks * COIN_BLOCK + tid, w.blocks, x);
  if (tid == 0) {
    w.part[(size_t)i * w.S + slice] = r;
    if (slice == 0) { w.key[i] = 0; w.arrived[i] = 0; }
  }
}

// What coin_draw tells thread 0 of each workgroup: nothing, that the drafted token stays (the workgroup of slice 0 says so), or
// the residual's token (the last workgroup; x if the residual is empty, which cannot occur when the coin fails).
enum CoinSays { COIN_NOTHING, COIN_KEPT, COIN_DRAWN };

template <bool ONE>
__device__ __forceinline__ CoinSays coin_draw(const float* __restrict__ lq, const float* __restrict__ lp, int V, float it,
                                              unsigned seed_lo, unsigned seed_hi, int b, int t, int x, const CoinWork& w, int i,
                                              int* drawn) {
  __shared__ u64 s_key[COIN_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, slice = blockIdx.y, first = slice * w.blocks * COIN_BLOCK + tid;
  CoinWords a;                                           // block 0: on its way while the coin is settled
  const float xq = lq[x], xp = lp[x];
  float mq = -INFINITY, mp = -INFINITY, sq = 0.f, sp = 0.f;
  if constexpr (ONE) {
    const float4 r = coin_sums(lq, lp, V, it, first, w.blocks, a);
    mq = r.x; mp = r.y; sq = r.z; sp = r.w;
  } else {
    a.load(lq, lp, first, V, it);
    const float4* part = w.part + (size_t)i * w.S;
    for (int s = lane; s < w.S; s += 64) { const float4 v = part[s]; mq = fmaxf(mq, v.x); mp = fmaxf(mp, v.y); }
    mq = wave_max(mq);
    mp = wave_max(mp);
    for (int s = lane; s < w.S; s += 64) {
      const float4 v = part[s];
      sq += v.z * expf(v.x - mq);
      sp += v.w * expf(v.y - mp);
    }
    sq = wave_sum(sq);
    sp = wave_sum(sp);
  }
  const float lse_q = mq + logf(sq), lse_p = mp + logf(sp);
  const float log_ratio = (xp * it - lse_p) - (xq * it - lse_q);
  const unsigned cw = philox_word(seed_lo, seed_hi, 2u, (unsigned)b, (unsigned)t, 0u);
  const float coin = ((float)(cw >> 9) + 0.5f) * 1.1920928955078125e-07f;
  if (coin <= fminf(1.0f, expf(log_ratio))) return slice == 0 ? COIN_KEPT : COIN_NOTHING;   // uniform over the workgroups
  u64 best = 0;
  for (int k = 0; k < w.blocks; ++k) {
    const int v0 = first + k * COIN_BLOCK;
    if (k) a.load(lq, lp, v0, V, it);
#pragma unroll
    for (int u = 0; u < COIN_U; ++u) {
      const int v = v0 + u * COIN_THREADS;
      const float r = expf(a.p[u] - lse_p) - expf(a.q[u] - lse_q);   // (0 beyond the vocabulary)
      if (r > 0.f) {
        const float z = logf(r) + gumbel_from_word(philox_word(seed_lo, seed_hi, 1u, (unsigned)b, (unsigned)t, (unsigned)v));
        best = umax64(best, pack_key(z, (unsigned)v));
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) best = umax64(best, shfl_xor_u64(best, o));
  if (lane == 0) s_key[tid >> 6] = best;
  __syncthreads();
  if (tid) return COIN_NOTHING;
#pragma unroll
  for (int q = 1; q < COIN_THREADS / 64; ++q) best = umax64(best, s_key[q]);
  if constexpr (!ONE) {
    atomicMax(w.key + i, best);
    // The key is there before the arrival; the two atomics are all that the workgroups share, so waiting is enough (with a
    // __threadfence, which writes the L2 cache back, 24 tokens of 50257 words took 18.4 us instead of 14.9).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (atomicAdd(w.arrived + i, 1) != w.S - 1) return COIN_NOTHING;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    best = atomicMax(w.key + i, 0ull);
  }
  *drawn = best ? key_index(best) : x;
  return COIN_DRAWN;
}

}  // namespace sprinter
