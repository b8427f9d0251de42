// The coin min(1, p(x) / q(x)) of one drafted token and, where it fails, the draw from the residual max(0, p - q): shared by the
// correction of rejected rows (k_control.hip) and the speculative-decoding windows (k_sd.hip).
#pragma once
#include "dev.h"

namespace sprinter {

constexpr int COIN_THREADS = 1024;

// fold(v) over a workgroup of COIN_THREADS, in every thread.  s: 16 floats of LDS that nothing else uses.
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

// One workgroup of COIN_THREADS per token.  q = softmax(lq * it), p = softmax(lp * it); sweeps over the vocabulary for the
// maxima, the sums of exponentials and - only where the coin fails - the Gumbel-max draw from max(0, p - q), taken on
// ln(p - q) + noise of the target stream.  float32 throughout.  Returns (uniform) whether x is kept; *drawn (thread 0) is the
// residual's token, x if the residual is empty (which cannot occur when the coin fails).
// A row is read by one compute unit, so the loads in flight bound it: 16 waves with 8 loads of each row per lane requested
// together: 81 us for 80 tokens of a 50257-word vocabulary, 54 for 16; 4 waves with one load waited for at a time: 254 and 174.
__device__ __forceinline__ bool coin_or_residual(const float* __restrict__ lq, const float* __restrict__ lp, int V, float it,
                                                 unsigned seed_lo, unsigned seed_hi, int b, int t, int x, int* drawn) {
  constexpr int U = 8, STEP = COIN_THREADS * U;
  __shared__ float s_fold[4][COIN_THREADS / 64];
  __shared__ u64 s_key[COIN_THREADS / 64];
  const int tid = threadIdx.x;
  float a[U], c[U];
  auto load = [&](int v0) {                              // logits / T of U words per thread; -inf beyond the vocabulary
#pragma unroll
    for (int u = 0; u < U; ++u) { const int v = min(v0 + u * COIN_THREADS, V - 1); a[u] = lq[v]; c[u] = lp[v]; }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = v0 + u * COIN_THREADS < V;
      a[u] = in ? a[u] * it : -INFINITY;
      c[u] = in ? c[u] * it : -INFINITY;
    }
  };
  float mq = -INFINITY, mp = -INFINITY, sq = 0.f, sp = 0.f;
  for (int v0 = tid; v0 < V; v0 += STEP) {
    load(v0);
#pragma unroll
    for (int u = 0; u < U; ++u) { mq = fmaxf(mq, a[u]); mp = fmaxf(mp, c[u]); }
  }
  mq = coin_fold<true>(mq, s_fold[0]);
  mp = coin_fold<true>(mp, s_fold[1]);
  for (int v0 = tid; v0 < V; v0 += STEP) {
    load(v0);
#pragma unroll
    for (int u = 0; u < U; ++u) { sq += expf(a[u] - mq); sp += expf(c[u] - mp); }
  }
  sq = coin_fold<false>(sq, s_fold[2]);
  sp = coin_fold<false>(sp, s_fold[3]);
  const float lse_q = mq + logf(sq), lse_p = mp + logf(sp);
  const float log_ratio = (lp[x] * it - lse_p) - (lq[x] * it - lse_q);
  const unsigned cw = philox_word(seed_lo, seed_hi, 2u, (unsigned)b, (unsigned)t, 0u);
  const float coin = ((float)(cw >> 9) + 0.5f) * 1.1920928955078125e-07f;
  if (coin <= fminf(1.0f, expf(log_ratio))) return true;   // uniform over the workgroup
  u64 best = 0;
  for (int v0 = tid; v0 < V; v0 += STEP) {
    load(v0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int v = v0 + u * COIN_THREADS;
      const float r = expf(c[u] - lse_p) - expf(a[u] - lse_q);   // (0 beyond the vocabulary)
      if (r > 0.f) {
        const float z = logf(r) + gumbel_from_word(philox_word(seed_lo, seed_hi, 1u, (unsigned)b, (unsigned)t, (unsigned)v));
        best = umax64(best, pack_key(z, (unsigned)v));
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) best = umax64(best, shfl_xor_u64(best, o));
  if ((tid & 63) == 0) s_key[tid >> 6] = best;
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int q = 1; q < COIN_THREADS / 64; ++q) best = umax64(best, s_key[q]);
    *drawn = best ? key_index(best) : x;
  }
  return false;
}

}  // namespace sprinter
