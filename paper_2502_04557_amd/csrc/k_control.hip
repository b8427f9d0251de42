// HIP kernels of the batched SPRINTER decode step for gfx950: the decisions of Alg. 2 (threshold, compaction,
// commit), prefill row lists, the full-prefix work list and the p/q correction of Sec. 2, Eq. (1).
#include "coin.h"
#include <algorithm>
#include <cstring>

namespace sprinter {

// ===================================================== commit of a step
// Thread b commits row b's token c: token history, cache lengths, outputs, and the next step's draft row descriptors.
__device__ __forceinline__ void commit_row(const FinishArgs& a, int b, int c, bool acc, int draft_tok, float score, long long g) {
  a.committed[b] = c;
  a.st.last_tok[b] = c;
  const int lq = a.st.len_q[b] + 1;
  a.st.len_q[b] = lq;
  if (!acc) {
    a.st.len_p[b] = a.ctx_mode == 1 ? lq : a.st.len_p[b] + 1;
    a.st.n_target_calls[b] += 1;
  }
  a.st.hist[(size_t)b * a.st.hist_stride + lq] = c;
  if (a.o_committed) a.o_committed[b] = c;
  if (a.n_tokens > 0 && g < a.n_tokens) {
    const size_t o = (size_t)b * a.n_tokens + (size_t)g;
    if (a.g_tok) a.g_tok[o] = c;
    if (a.g_accept) a.g_accept[o] = acc ? 1 : 0;
    if (a.g_score) a.g_score[o] = score;
    if (a.g_draft_tok) a.g_draft_tok[o] = draft_tok;
  }
  a.d_b[b] = b;                                      // the next step's draft forward: every row, its last token at the next position
  a.d_tok[b] = c;
  a.d_pos[b] = lq;
  a.d_slot[b] = lq;
}
__device__ __forceinline__ void commit_counters(const FinishArgs& a, int R, long long g) {
  *a.d_n_rows = a.B;
  a.st.counters[0] += 1;
  a.st.counters[1] += (R > 0) ? 1 : 0;
  a.st.counters[2] += R;
  a.st.counters[3] = g + 1;
}

// ====================================== decide: arg-max merge, threshold, compaction
// Single workgroup of 1024 threads (B <= 1024).  accept <=> sigmoid(logit) >= tau in float32.
// Rejected rows are listed in ascending order: ballot + popcount inside each wave,
// wave totals prefix-summed through LDS.  A step without rejections is committed right here (f), so its chain ends with
// this launch.
__global__ __launch_bounds__(1024) void k_draft_decide(DecideArgs a, FinishArgs f, int row_lanes) {
  __shared__ int s_tok[1024];
  __shared__ int s_wave_cnt[16];
  __shared__ int s_rej[1024];
  __shared__ u64 s_key[16][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int B = a.B;
  // Arg-max merge over the LM head's per-workgroup partials part[workgroup][row]: row_lanes (a power of two, min(B, 64)
  // rounded up) lanes of a wave take consecutive rows of one workgroup (with a lane per workgroup every 8-byte load hit its
  // own cache line: 37 us at 64 rows and 512 workgroups), the wave's 64 / row_lanes groups and the 16 waves different
  // workgroups, eight loads in flight per lane; then shuffles and LDS merge them.  At one row the whole merge is a single
  // round of loads (with one active lane per wave it took four rounds, and with keys 32 KiB apart as many TLB misses:
  // kernel 7.6 us at one row and 393 workgroups, now 5.2).
  float z = 0.f;                                     // the verifier's output logit: offset + the hidden chunks' shares, in order
  if (tid < B) {                                     // (requested ahead of the merge below)
    z = a.b2[0];
#pragma unroll 8
    for (int c = 0; c < a.n_chunks; ++c) z += a.ver_part[(size_t)c * B + tid];
  }
  const int rl = lane & (row_lanes - 1), subs = 64 / row_lanes, first = w * subs + lane / row_lanes, stride = 16 * subs;
  for (int rb = 0; rb < B; rb += row_lanes) {
    const int m = rb + rl;
    u64 k = 0;
    if (m < B)
      for (int i0 = first; i0 < a.n_lm_wg; i0 += 8 * stride) {
        u64 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = i0 + stride * u;
          v[u] = i < a.n_lm_wg ? a.am_part[(size_t)i * a.Mpad + m] : 0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) k = umax64(k, v[u]);
      }
    for (int o = row_lanes; o < 64; o <<= 1) k = umax64(k, shfl_xor_u64(k, o));
    s_key[w][lane] = k;
    __syncthreads();
    if (tid < row_lanes && m < B) {
      u64 kk = s_key[0][lane];
#pragma unroll
      for (int q = 1; q < 16; ++q) kk = umax64(kk, s_key[q][lane]);
      s_tok[m] = key_index(kk);
    }
    __syncthreads();
  }
  bool active = tid < B;
  float score = 0.f;
  bool acc = true;
  if (active) {
    score = 1.0f / (1.0f + expf(-z));
    acc = score >= *a.tau_ptr;
  }
  const bool rej = active && !acc;
  const u64 mask = __ballot(rej);
  const int rank = __popcll(mask & ((1ull << lane) - 1ull));
  if (lane == 0) s_wave_cnt[w] = __popcll(mask);
  __syncthreads();
  int off = 0, total = 0;
  for (int q = 0; q < 16; ++q) {
    int c = s_wave_cnt[q];
    if (q < w) off += c;
    total += c;
  }
  if (tid == 0 && total == 0 && a.host_word) {       // the host may queue the next step while this kernel commits
    if (a.ctx_mode == 1) a.host_word[1] = 0;
    __hip_atomic_store(a.host_word, (unsigned long long)a.ticket << 32, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (rej) s_rej[off + rank] = tid;
  const int dt = active ? s_tok[tid] : 0;
  if (active) {
    a.draft_tok[tid] = dt;
    a.score[tid] = score;
    a.accept[tid] = acc ? 1 : 0;
    a.committed[tid] = acc ? dt : -1;
    if (a.o_draft_tok) a.o_draft_tok[tid] = dt;
    if (a.o_score) a.o_score[tid] = score;
    if (a.o_accept) a.o_accept[tid] = acc ? 1 : 0;
  }
  if (total == 0) {
    const long long g = a.st.counters[3];
    __syncthreads();                                 // (everybody has read the generation index)
    if (active) commit_row(f, tid, dt, true, dt, score, g);
    if (tid == 0) {
      *a.n_rej = 0;
      *a.t_n_rows = 0;
      if (a.o_n_rej) *a.o_n_rej = 0;
      commit_counters(f, 0, g);
    }
    return;
  }
  __syncthreads();
  if (tid < total) {
    int b = s_rej[tid];
    a.rej_idx[tid] = b;
    if (a.o_rej_idx) a.o_rej_idx[tid] = b;
    a.t_b[tid] = b;
    a.t_tok[tid] = a.st.last_tok[b];
    a.t_pos[tid] = a.st.len_q[b];       // true position id of the input token
    a.t_slot[tid] = a.st.len_p[b];      // next free slot of the row's target cache
  }
  if (a.ctx_mode == 1) {
    // work list of the full-prefix target pass: entries per rejected row, exclusive prefix sums in ascending row order
    __syncthreads();
    int cnt = 0;
    if (tid < total) { const int b = s_rej[tid]; cnt = a.st.len_q[b] - a.st.len_p[b] + 1; }
    int inc = cnt;                                     // inclusive scan inside the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const int up = __shfl_up(inc, o); if (lane >= o) inc += up; }
    if (lane == 63) s_wave_cnt[w] = inc;
    __syncthreads();
    int before = 0, all = 0;
    for (int q = 0; q < 16; ++q) { const int c = s_wave_cnt[q]; if (q < w) before += c; all += c; }
    if (tid < total) a.ent_off[tid] = before + inc - cnt;
    if (tid == 0) {
      a.ent_off[total] = all;
      if (a.host_word) a.host_word[1] = (unsigned long long)(unsigned)all;   // ordered before the release store below
    }
  }
  if (tid == 0) {
    *a.n_rej = total;
    *a.t_n_rows = total;
    if (a.o_n_rej) *a.o_n_rej = total;
    if (a.host_word)    // one 8-byte store into pinned host memory: the host launches the target pass from it
      __hip_atomic_store(a.host_word, ((unsigned long long)a.ticket << 32) | (unsigned)total, __ATOMIC_RELEASE,
                         __HIP_MEMORY_SCOPE_SYSTEM);
  }
}
void launch_draft_decide(const DecideArgs& a, const FinishArgs& f, hipStream_t s) {
  int row_lanes = 1;
  while (row_lanes < a.B && row_lanes < 64) row_lanes <<= 1;
  hipLaunchKernelGGL(k_draft_decide, dim3(1), dim3(1024), 0, s, a, f, row_lanes);
}

// ===================== finish: target arg-max merge, scatter back, advance state
__global__ __launch_bounds__(1024) void k_step_finish(FinishArgs a) {
  __shared__ int s_commit[1024];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int B = a.B, R = *a.n_rej;
  if (tid < B) s_commit[tid] = a.committed[tid];
  __syncthreads();
  if (!a.pre_merged) {
    for (int i = w; i < R; i += 16) {
      u64 k = merge_partials(a.am_part, a.n_lm_wg, a.Mpad, i, lane);
      if (lane == 0) s_commit[a.rej_idx[i]] = key_index(k);
    }
  }
  const long long g = a.st.counters[3];
  __syncthreads();
  if (tid < B) commit_row(a, tid, s_commit[tid], a.accept[tid] != 0, a.draft_tok[tid], a.score[tid], g);
  if (tid == 0) commit_counters(a, R, g);
}
void launch_step_finish(const FinishArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_step_finish, dim3(1), dim3(1024), 0, s, a);
}

// ================================================================ prefill
// Chunked prefill: the prompts go into the token history, every row's caches count as empty and every row is
// listed, so that the full-prefix work-list kernel (k_catchup_chunk) enumerates the prompt positions 0 .. P_b-2
// in row-major order from the prefix sums the host uploaded.
// One workgroup per row (one thread per row copied its prompt token after token: 1.1 ms for 2000 tokens).
__global__ __launch_bounds__(256) void k_prefill_begin(const int* __restrict__ prompt, int max_prompt, int B, State st,
                                                       int* rej_idx, int* n_rej) {
  const int b = blockIdx.x, P = st.prompt_len[b];
  for (int j = threadIdx.x; j < P; j += 256) st.hist[(size_t)b * st.hist_stride + j] = prompt[(size_t)b * max_prompt + j];
  if (threadIdx.x == 0) {
    st.len_p[b] = 0;
    rej_idx[b] = b;
    if (b == 0) *n_rej = B;
  }
}
void launch_prefill_begin(const int* prompt, int max_prompt, int B, State st, int* rej_idx, int* n_rej, hipStream_t s) {
  hipLaunchKernelGGL(k_prefill_begin, dim3(B), dim3(256), 0, s, prompt, max_prompt, B, st, rej_idx, n_rej);
}

__global__ __launch_bounds__(1024) void k_prefill_finish(const int* __restrict__ prompt, int max_prompt, int B,
                                                         State st, int* d_n_rows, int* d_b, int* d_tok, int* d_pos,
                                                         int* d_slot) {
  const int tid = threadIdx.x;
  if (tid < B) {
    int P = st.prompt_len[tid];
    int last = prompt[(size_t)tid * max_prompt + P - 1];
    st.last_tok[tid] = last;
    st.len_q[tid] = P - 1;
    st.len_p[tid] = P - 1;
    st.n_target_calls[tid] = 0;
    d_b[tid] = tid;
    d_tok[tid] = last;
    d_pos[tid] = P - 1;
    d_slot[tid] = P - 1;
  }
  if (tid == 0) {
    *d_n_rows = B;
    st.counters[0] = st.counters[1] = st.counters[2] = st.counters[3] = 0;
  }
}
void launch_prefill_finish(const int* prompt, int max_prompt, int B, State st, int* d_n_rows, int* d_b, int* d_tok,
                           int* d_pos, int* d_slot, hipStream_t s) {
  hipLaunchKernelGGL(k_prefill_finish, dim3(1), dim3(1024), 0, s, prompt, max_prompt, B, st, d_n_rows, d_b, d_tok,
                     d_pos, d_slot);
}

// ============================================ full-prefix target context: work list
// One thread per entry of the chunk: binary search of the entry's rejected row in the prefix sums.
__global__ __launch_bounds__(1024) void k_catchup_chunk(CatchupArgs a) {
  const int R = *a.n_rej;
  for (int i = threadIdx.x; i < a.n; i += 1024) {
    const int e = a.start + i;
    int lo = 0, hi = R - 1;                            // last row index with ent_off[row] <= e
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.ent_off[mid] <= e) lo = mid; else hi = mid - 1;
    }
    const int b = a.rej_idx[lo];
    const int pos = a.st.len_p[b] + (e - a.ent_off[lo]);
    a.t_b[i] = b;
    a.t_tok[i] = a.st.hist[(size_t)b * a.st.hist_stride + pos];
    a.t_pos[i] = pos;
    a.t_slot[i] = pos;                                 // in this mode the target cache has no gaps: slot = position
    a.t_last[i] = (e + 1 == a.ent_off[lo + 1]) ? 1 : 0;
  }
  if (threadIdx.x == 0) *a.t_n_rows = a.n;
}
void launch_catchup_chunk(const CatchupArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_catchup_chunk, dim3(1), dim3(1024), 0, s, a);
}

__global__ __launch_bounds__(256) void k_catchup_collect(const u64* __restrict__ am_part, int n_lm_wg, int Mpad,
                                                        const int* __restrict__ n_rows, const int* __restrict__ t_b,
                                                        const int* __restrict__ t_last, int* __restrict__ committed) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wave_index();
  if (i >= *n_rows || !t_last[i]) return;
  const u64 k = merge_partials(am_part, n_lm_wg, Mpad, i, lane);
  if (lane == 0) committed[t_b[i]] = key_index(k);
}
void launch_catchup_collect(const unsigned long long* am_part, int n_lm_wg, int Mpad, const int* n_rows, const int* t_b,
                            const int* t_last, int* committed, int max_rows, hipStream_t s) {
  hipLaunchKernelGGL(k_catchup_collect, dim3((max_rows + 3) / 4), dim3(256), 0, s, am_part, n_lm_wg, Mpad, n_rows, t_b,
                     t_last, committed);
}

// ===================================== rejection by p/q coin + residual (Sec. 2, Eq. (1))
// w.S workgroups per row of the target pass (coin.h).
__device__ __forceinline__ bool corrected(const SdArgs& a, int i) { return i < *a.n_rows && !(a.t_last && !a.t_last[i]); }

__global__ __launch_bounds__(COIN_THREADS) void k_sd_correct_sums(SdArgs a, CoinWork w) {
  const int i = blockIdx.x;
  if (corrected(a, i)) coin_slice(a.dl + (size_t)a.t_b[i] * a.V, a.tl + (size_t)i * a.V, a.V, a.inv_temperature, w, i);
}
template <bool ONE>
__global__ __launch_bounds__(COIN_THREADS) void k_sd_correct(SdArgs a, CoinWork w) {
  const int i = blockIdx.x;
  if (!corrected(a, i)) return;
  const int b = a.t_b[i], t = a.t_pos[i] + 1, x = a.draft_tok[b], V = a.V;
  int drawn = 0;
  const CoinSays say = coin_draw<ONE>(a.dl + (size_t)b * V, a.tl + (size_t)i * V, V, a.inv_temperature, a.seed_lo, a.seed_hi, b, t, x,
                                 w, i, &drawn);
  if (threadIdx.x == 0 && say != COIN_NOTHING) {
    a.committed[b] = say == COIN_KEPT ? x : drawn;
    if (say == COIN_KEPT) atomicAdd(a.coin_kept, 1);
  }
}
void launch_sd_correct(const SdArgs& a, int max_rows, void* work, size_t work_bytes, hipStream_t s) {
  const CoinWork w = coin_work(work, work_bytes, max_rows, a.V);
  if (w.S == 1) {
    hipLaunchKernelGGL(k_sd_correct<true>, dim3(max_rows), dim3(COIN_THREADS), 0, s, a, w);
    return;
  }
  hipLaunchKernelGGL(k_sd_correct_sums, dim3(max_rows, w.S), dim3(COIN_THREADS), 0, s, a, w);
  hipLaunchKernelGGL(k_sd_correct<false>, dim3(max_rows, w.S), dim3(COIN_THREADS), 0, s, a, w);
}

__global__ void k_set_i32(int* p, int v) { *p = v; }
void launch_set_i32(int* p, int v, hipStream_t s) { hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, s, p, v); }

__global__ void k_set_f32(float* p, float v) { *p = v; }
void launch_set_f32(float* p, float v, hipStream_t s) { hipLaunchKernelGGL(k_set_f32, dim3(1), dim3(1), 0, s, p, v); }

__global__ void k_reset_gen_idx(long long* counters) { counters[3] = 0; }
void launch_reset_gen_idx(long long* counters, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_gen_idx, dim3(1), dim3(1), 0, s, counters);
}

__global__ __launch_bounds__(256) void k_copy_rows(const float* __restrict__ src, float* __restrict__ dst,
                                                   const int* __restrict__ n_rows, int row_len) {
  int r = blockIdx.x;
  if (r >= *n_rows) return;
  for (int k = threadIdx.x; k < row_len; k += 256) dst[(size_t)r * row_len + k] = src[(size_t)r * row_len + k];
}
void launch_copy_f32(const float* src, float* dst, const int* n_rows, int row_len, int max_rows, hipStream_t s) {
  hipLaunchKernelGGL(k_copy_rows, dim3(max_rows), dim3(256), 0, s, src, dst, n_rows, row_len);
}

}  // namespace sprinter
