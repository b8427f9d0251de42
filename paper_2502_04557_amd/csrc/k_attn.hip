// HIP kernels of the batched SPRINTER decode step for gfx950: single-query attention over the KV caches.
#include "dev.h"
#include <algorithm>
#include <cstring>

namespace sprinter {

// ============================================================== attention
// One workgroup per (row, KV head): rotary on q and the new k, append k/v to the
// cache, scores against all cached keys, softmax, weighted sum of values.
// The G query heads that share the KV head are processed together.
struct AttnArgs {
  const float* y; const float* rope; RowDesc rd;
  void* kcache; void* vcache; size_t layer_off;
  int H, KVH, G, lg, dqkv, max_seq, use_rope; float scale;   // G = H / KVH = 1 << lg
  void* ao; int ao_K;
  float* split;   // k_attn_dec_bf16 with several workgroups per row and KV head: partial results [row][KV head][z][query head][DH + 2]
  int phase;   // 0 append + attend, 1 append only, 2 attend only, 3 attend only over long runs of one row (launcher only)
};

// The kernels of decode steps take what they use of it as single arguments, what they need first in front (internal.h); their caches are those of the layer.
#define ATTN_ARGS const float *y_, const int *b_, const int *slot_, void *kcache_, void *vcache_, int H_, int KVH_, int S_, int extra_, const int *n_rows_, void *ao_, const float *rope_
#define ATTN_VALUES(a, extra, S) (a).y, (a).rd.b, (a).rd.slot, (void*)((char*)(a).kcache + (a).layer_off * (S)), (void*)((char*)(a).vcache + (a).layer_off * (S)), (a).H, (a).KVH, (a).max_seq, extra, (a).rd.n_rows, (a).ao, (a).rope
template <int DH>
__device__ __forceinline__ AttnArgs attn_args(ATTN_ARGS, float* split) {
  AttnArgs a;
  a.y = y_; a.rd.b = b_; a.rd.slot = slot_; a.rd.n_rows = n_rows_; a.kcache = kcache_; a.vcache = vcache_; a.layer_off = 0; a.rope = rope_;
  a.H = H_; a.KVH = KVH_; a.dqkv = (H_ + 2 * KVH_) * DH; a.max_seq = S_; a.ao = ao_; a.ao_K = H_ * DH; a.split = split; a.phase = extra_;
  a.scale = DH == 64 ? 0.125f : 0x1.6a09e6p-4f;                  // 1.0f / sqrtf(DH)
  return a;
}

// float32 mode.  One workgroup of four waves per (row, KV head), which attends for the G query heads that share the KV head in one pass
// over the cached keys.  A key is a DPP row of 16 lanes, each with DH / 16 consecutive columns; a wave takes blocks of 32 keys - 8 per
// DPP row - whose keys and values are requested together.  Every DPP row is a stream of its own with its maximum, sum and
// output columns, so nothing crosses rows or waves before the end, where LDS merges the 16 streams.  Queries, new key and new
// value are computed from the projection by every wave in the layout it uses them in, without LDS.
// What bounds it is latency: arguments, then descriptors and projection, then keys and values, then about 200 vector instructions per
// block.  us per launch, of a kernel with one pass over the keys for the scores, one for the values and barriers and shuffles through
// LDS in between -> of this one: heads of 64, 1 row of 40 keys 4.5 -> 3.4, 6 rows x 8 heads x 60 keys 6.6 -> 4.1, 24 x 8 x 90 10.9 -> 5.3; of 128,
// 3 x 8 x 300 43.6 -> 11.2, 8 heads per KV head, 2 x 2 x 500 138 -> 39.
// Sums are taken in pairs - a block's weights and values before they join the stream's, the 16 streams at the end - since a stream has a
// maximum, and a factor, of its own.  Error against 64 bits (2-norm over the result's, mean of 24 sets of 16 rows), one maximum per row
// -> in order -> in pairs: 64 columns, 16 - 60 keys 1.24e-7 -> 1.27e-7 -> 1.21e-7, 60 - 130 1.37e-7 -> 1.51e-7 -> 1.32e-7, 130 - 300 1.51e-7 ->
// 1.66e-7 -> 1.42e-7; 128 columns, 60 - 130 1.46e-7 -> 1.59e-7 -> 1.44e-7; it costs 0.05 - 0.09 us of 3.6 - 13.4 us per launch.
template <int DH, int G, bool ROPE>
__global__ __launch_bounds__(256) void k_attn_f32(ATTN_ARGS) {   // extra: phase
  const AttnArgs a = attn_args<DH>(y_, b_, slot_, kcache_, vcache_, H_, KVH_, S_, extra_, n_rows_, ao_, rope_, nullptr);
  constexpr int E = DH / 16, Q4 = E / 4, NK = 8, KB = 4 * NK, HALF = DH / 2;   // columns per lane, float4s of them, keys per stream and block
  __shared__ float s_m[16][G], s_l[16][G];
  __shared__ __attribute__((aligned(16))) float s_o[16][G][DH];
  const int r = blockIdx.y, kvh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = wave_index(), l16 = lane & 15, lq = lane >> 4;
  const int n_rows = *a.rd.n_rows, b = a.rd.b[r], slot = a.rd.slot[r], S = a.max_seq;   // (the lists hold every row the grid covers)
  const float* __restrict__ y = a.y + (size_t)r * a.dqkv;
  const int d0 = l16 * E, p0 = d0 ^ HALF;
  const float* __restrict__ yk = y + (size_t)(a.H + kvh) * DH;
  const float* __restrict__ yv = y + (size_t)(a.H + a.KVH + kvh) * DH;
  float q[G][E], kn[E], vn[E];
  {
    float qp[G][E], kp[E], cs[2 * E];
    auto load = [&](float (&x)[E], const float* p) {
#pragma unroll
      for (int i = 0; i < Q4; ++i) *reinterpret_cast<float4*>(&x[4 * i]) = reinterpret_cast<const float4*>(p)[i];
    };
#pragma unroll
    for (int g = 0; g < G; ++g) {
      load(q[g], y + (size_t)(kvh * G + g) * DH + d0);
      if (ROPE) load(qp[g], y + (size_t)(kvh * G + g) * DH + p0);
    }
    load(kn, yk + d0);
    load(vn, yv + d0);
    if (ROPE) {
      load(kp, yk + p0);
      const float4* c4 = reinterpret_cast<const float4*>(a.rope + (size_t)r * DH + 2 * (d0 % HALF));
#pragma unroll
      for (int i = 0; i < 2 * Q4; ++i) *reinterpret_cast<float4*>(&cs[4 * i]) = c4[i];
    }
    if (r >= n_rows) return;
    const bool upper = d0 >= HALF;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (ROPE) {
        const float c = cs[2 * e], sn = cs[2 * e + 1];
#pragma unroll
        for (int g = 0; g < G; ++g) q[g][e] = (upper ? q[g][e] * c + qp[g][e] * sn : q[g][e] * c - qp[g][e] * sn) * a.scale;
        kn[e] = upper ? kn[e] * c + kp[e] * sn : kn[e] * c - kp[e] * sn;
      } else {
#pragma unroll
        for (int g = 0; g < G; ++g) q[g][e] *= a.scale;
      }
    }
  }
  float* __restrict__ Kc = (float*)a.kcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH + d0;
  float* __restrict__ Vc = (float*)a.vcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH + d0;
  if (a.phase != 2 && tid < 16) {
#pragma unroll
    for (int i = 0; i < Q4; ++i) {
      reinterpret_cast<float4*>(Kc + (size_t)slot * DH)[i] = *reinterpret_cast<const float4*>(&kn[4 * i]);
      reinterpret_cast<float4*>(Vc + (size_t)slot * DH)[i] = *reinterpret_cast<const float4*>(&vn[4 * i]);
    }
  }
  if (a.phase == 1) return;
  float m[G], l[G], o[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY; l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) o[g][e] = 0.f;
  }
  for (int kb = w * KB; kb <= slot; kb += 4 * KB) {              // (scalar) key of stream lq: kb + 4 j + lq
    float k[NK][E], v[NK][E];
#pragma unroll
    for (int j = 0; j < NK; ++j)
#pragma unroll
      for (int i = 0; i < Q4; ++i) {
        const size_t off = (size_t)min(kb + 4 * j + lq, slot) * DH;
        *reinterpret_cast<float4*>(&k[j][4 * i]) = reinterpret_cast<const float4*>(Kc + off)[i];
        *reinterpret_cast<float4*>(&v[j][4 * i]) = reinterpret_cast<const float4*>(Vc + off)[i];
      }
    if (kb + KB > slot) {                                        // (scalar) the row's last block: its own key and value, which the cache may not hold yet
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        const int behind = kb + 4 * j + lq - slot;               // > 0: no key (its score is masked below; 0 x its value has to be 0)
#pragma unroll
        for (int e = 0; e < E; ++e) { k[j][e] = behind >= 0 ? kn[e] : k[j][e]; v[j][e] = behind > 0 ? 0.f : behind == 0 ? vn[e] : v[j][e]; }
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float s[NK], mx = m[g];
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        float d = q[g][0] * k[j][0];
#pragma unroll
        for (int e = 1; e < E; ++e) d += q[g][e] * k[j][e];
        s[j] = kb + 4 * j + lq <= slot ? group_sum<16>(d) : -INFINITY;
        mx = fmaxf(mx, s[j]);
      }
      if (kb + lq <= slot) {                                     // (the same in a stream's 16 lanes) it has a key in this block
        const float off = mx == -INFINITY ? 0.f : mx;            // (all its scores so far are -inf: weights of 0, as in a row with one maximum)
        const float corr = expf(m[g] - off);
        m[g] = mx;
        static_assert(NK == 8, "the sum below");
        float p[NK];
#pragma unroll
        for (int j = 0; j < NK; ++j) p[j] = expf(s[j] - off);
        l[g] = l[g] * corr + (((p[0] + p[4]) + (p[2] + p[6])) + ((p[1] + p[5]) + (p[3] + p[7])));
#pragma unroll
        for (int e = 0; e < E; ++e) {
          float even = p[0] * v[0][e], odd = p[1] * v[1][e];
#pragma unroll
          for (int j = 2; j < NK; j += 2) { even += p[j] * v[j][e]; odd += p[j + 1] * v[j + 1][e]; }
          o[g][e] = o[g][e] * corr + (even + odd);
        }
      }
    }
  }
  const int st = w * 4 + lq;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    if (l16 == 0) { s_m[st][g] = m[g]; s_l[st][g] = l[g]; }
#pragma unroll
    for (int i = 0; i < Q4; ++i) *reinterpret_cast<float4*>(&s_o[st][g][d0 + 4 * i]) = *reinterpret_cast<const float4*>(&o[g][4 * i]);
  }
  __syncthreads();
  for (int idx = tid; idx < G * DH; idx += 256) {
    const int g = idx / DH, i = idx % DH;
    float mx = s_m[0][g], den[16], num[16];                      // (stream 0 has key 0)
#pragma unroll
    for (int t = 1; t < 16; ++t) mx = fmaxf(mx, s_m[t][g]);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const float c = expf(s_m[t][g] - mx);
      den[t] = c * s_l[t][g];
      num[t] = c * s_o[t][g][i];
    }
#pragma unroll
    for (int h = 8; h; h >>= 1)
#pragma unroll
      for (int t = 0; t < h; ++t) { den[t] += den[t + h]; num[t] += num[t + h]; }
    act_store<float>((float*)a.ao, r, kvh * G * DH + idx, a.ao_K, num[0] / den[0]);
  }
}

// A value tile's operand piece is 8 consecutive keys of one column, two a register: masks of its first n keys.  The keys beyond a
// row's last one are cleared with them (the cache may hold anything there, and 0 x NaN is NaN on the matrix cores).
__device__ __forceinline__ void vt_first(int n, unsigned (&keep)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) keep[e] = n > 2 * e + 1 ? 0xffffffffu : n > 2 * e ? 0xffffu : 0u;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding global access
// of the wave (vmcnt(0)): here that would be the first block's keys and values, requested on purpose long before
// they are needed, and the cache append.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// bf16 single-query attention on the matrix cores: one workgroup of NW waves per (row, KV head); the G query heads
// that share the KV head are rows of one 16-row operand, so a cached key costs the same whatever G is and the
// kernel is left with streaming the cache.  Wave w takes the 32-key blocks w, w + NW, ...; per block
// S = Q K^T (Q rotated, scaled and split into hi + lo bf16 planes in LDS, so it enters at float32
// precision; K fragments straight from the cache), online softmax in float32 on the accumulator layout (the 16 keys
// of a tile sit in one DPP row), P through a wave-private piece of LDS into operand layout (hi + lo), V^T tiles
// straight from the cache, O += P V.  A block's keys and value tiles are requested a whole step ahead (two register
// buffers; the query operand is kept in LDS to make room); nothing in the loop synchronises waves.  The row's own key and value
// (the token being processed) are computed in the prologue, appended to the cache by the waves that prepared them and patched from
// LDS into the operands of the block that holds slot `slot`, which is the row's last block; keys beyond it are masked.
// What bounds a short context is the wave's own instructions: alone on its SIMD it issues one every 4 - 5 cycles.  Operand row 4 j + v
// therefore holds head j NV + v (NV = 1 up to four heads, 2 for eight; the rows between repeat a head), so that the softmax of an
// accumulator is done for NV registers instead of four: 2450 -> 790 cycles per step at 64 columns and one head.  us per launch in a chain,
// with that, with the masks of the last block in two instructions a register and with loads only in the waves that use them: heads of 64,
// 150 keys, 25 of them: 6 rows 6.15 -> 5.08, 16 rows 8.4 -> 7.5; 60 keys, 1 row 4.7 -> 3.1; of 128, 300 keys, 32: 3 rows 10.5 -> 8.7, 33 rows (162
// MB) 41.9 -> 36.4; 8 KV heads, 540 keys, 17 rows 16.9 -> 13.1.  Long contexts and many rows: the cache, at 4.3 - 4.8 TB/s.  (When eight waves: at the launch.)
// The waves' partial results are merged through LDS at the end.  gridDim.z = extra > 1: that many workgroups share the keys (their waves
// count on), each leaves its unnormalised result, maximum and sum in a.split, and k_attn_merge puts them together.
template <int DH, int NW, int NV, bool ROPE>
__global__ __launch_bounds__(NW * 64, 2) void k_attn_dec_bf16(ATTN_ARGS, float* split_) {   // extra: workgroups per row and KV head
  const AttnArgs a = attn_args<DH>(y_, b_, slot_, kcache_, vcache_, H_, KVH_, S_, extra_, n_rows_, ao_, rope_, split_);
  constexpr int T = DH / 32, CT = DH / 16, PS = 36, HALF = DH / 2, GMAX = 4 * NV;
  constexpr float NEG = -1e30f;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) float lds_p[NW][GMAX * PS];
  __shared__ __attribute__((aligned(16))) bf16_t lds_kn[DH], lds_vn[DH];
  __shared__ uint4 lds_q[2][T][64];
  __shared__ float s_ml[NW][GMAX][2];
  __shared__ float s_o[NW][GMAX][DH];
  const int r = blockIdx.y;
  const int kvh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = wave_index();
  const int l16 = lane & 15, lq = lane >> 4, G = H_ / KVH_;
  const int n_rows = *a.rd.n_rows, b = a.rd.b[r], slot = a.rd.slot[r], S = a.max_seq;   // (the lists hold every row the grid covers)
  const int op_head = min((l16 >> 2) * NV + min(l16 & 3, NV - 1), G - 1);               // the head that operand row l16 holds
  // What depends on the row index alone is requested first, before the row's descriptor is known (the projection buffer holds
  // every row the grid covers): wave t < T takes the 32-column piece t of the query heads and of the new key, with their rotary
  // partners and angles, wave VW the new value; the others request nothing here (a load costs the compute unit's address unit 16
  // cycles whether its data are dropped or not).
  constexpr int VW = T < NW ? T : NW - 1;
  const float* __restrict__ y = a.y + (size_t)r * a.dqkv;
  const float* __restrict__ rp = a.rope + (size_t)r * DH;
  const float* __restrict__ yq = y + (size_t)(kvh * G + op_head) * DH;
  const float* __restrict__ yk = y + (size_t)(a.H + kvh) * DH;
  const float* __restrict__ yv = y + (size_t)(a.H + a.KVH + kvh) * DH;
  const int d0 = w * 32 + lq * 8, p0 = d0 ^ HALF;
  float x[8], xp[8], kx[8], kp[8], cs[16], vraw[DH / 64];
  if (w < T) {                                                   // (scalar)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *reinterpret_cast<float4*>(&x[4 * i]) = reinterpret_cast<const float4*>(yq + d0)[i];
      *reinterpret_cast<float4*>(&kx[4 * i]) = reinterpret_cast<const float4*>(yk + d0)[i];
      if (ROPE) {
        *reinterpret_cast<float4*>(&xp[4 * i]) = reinterpret_cast<const float4*>(yq + p0)[i];
        *reinterpret_cast<float4*>(&kp[4 * i]) = reinterpret_cast<const float4*>(yk + p0)[i];
      }
    }
    if (ROPE) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(&cs[4 * i]) = reinterpret_cast<const float4*>(rp + 2 * (d0 % HALF))[i];
    }
  }
  if (w == VW) {
#pragma unroll
    for (int i = 0; i < DH / 64; ++i) vraw[i] = yv[i * 64 + lane];
  }
  if (r >= n_rows) return;
  bf16_t* __restrict__ Kc = (bf16_t*)a.kcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH;
  bf16_t* __restrict__ Vc = (bf16_t*)a.vcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH;
  const int wz = blockIdx.z * NW + w, NZ = extra_ * NW;          // this wave among all that share the keys
  const int n_steps = (slot + 32 * NZ) / (32 * NZ);             // blocks 0 .. slot / 32, NZ per step
  // Two register buffers: a block's key fragments and value tiles are requested a whole step ahead (the query
  // operand lives in LDS to make room for them).
  // A block beyond the row's last one (a last step has up to NZ - 1, and the loop requests a step more than it uses) is fully masked.
  // At 128 columns it is requested from buffers of no length (a scalar choice): zeros, and the compute unit pulls nothing, where
  // reading the last block again took its share of 48 KB/us (heads of 128, 300 keys, 32 of them: 33 rows 39.0 -> 36.4 us, 59 rows 62.2 -> 59.2;
  // 8 KV heads, 540 keys, 17 rows 14.3 -> 13.1).  At 64 columns the descriptors cost few workgroups as much as the loads (25 heads, 150
  // keys, 6 rows 4.9 / 5.2; 8 KV heads, 1800 keys, 4 rows 8.3 / 8.8; but 25 heads, 16 rows 7.5 / 7.0): the last one again, a scalar clamp.
  // Inside a block nothing is clamped: the caches hold a multiple of 32 slots per (row, KV head), so every key of a block that
  // exists lies inside the cache.  Per-lane addresses or offsets once, block offsets are scalars.
  struct Blk { u32x4 k[2][T]; u32x4 v[CT]; };
  const int k_lane = l16 * DH + lq * 8, v_lane = lane * 8;       // elements
  const bf16_t *const k_ptr = Kc + k_lane, *const v_ptr = Vc + v_lane;
  const int kb_last = slot & ~31;
  auto fetch = [&](Blk& B, int kb) {
    if constexpr (DH == 128) {
      const bool in = kb <= kb_last;
      const int bytes = in ? 32 * DH * 2 : 0;                    // of a block's keys, and of its value tiles
      const size_t off = (size_t)(in ? kb : 0) * DH;
      const auto kr = __builtin_amdgcn_make_buffer_rsrc(Kc + off, 0, bytes, 0x00020000);
      const auto vr = __builtin_amdgcn_make_buffer_rsrc(Vc + off, 0, bytes, 0x00020000);
#pragma unroll
      for (int tile = 0; tile < 2; ++tile)
#pragma unroll
        for (int t = 0; t < T; ++t)
          B.k[tile][t] = __builtin_amdgcn_raw_buffer_load_b128(kr, 2 * (k_lane + tile * 16 * DH + t * 32), 0, 0);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) B.v[ct] = __builtin_amdgcn_raw_buffer_load_b128(vr, 2 * (v_lane + ct * 512), 0, 0);
    } else {
      const size_t off = (size_t)min(kb, kb_last) * DH;          // elements; the same for keys and value tiles
#pragma unroll
      for (int tile = 0; tile < 2; ++tile)
#pragma unroll
        for (int t = 0; t < T; ++t) B.k[tile][t] = *reinterpret_cast<const u32x4*>(k_ptr + off + tile * 16 * DH + t * 32);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) B.v[ct] = *reinterpret_cast<const u32x4*>(v_ptr + off + ct * 512);
    }
  };
  Blk A, B;
  fetch(A, wz * 32);
  if (w < T) {
    const bool upper = d0 >= HALF;
    float qv[8], kn[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (ROPE) {
        const float c = cs[2 * i], sn = cs[2 * i + 1];
        qv[i] = (upper ? x[i] * c + xp[i] * sn : x[i] * c - xp[i] * sn) * a.scale;
        kn[i] = upper ? kx[i] * c + kp[i] * sn : kx[i] * c - kp[i] * sn;
      } else {
        qv[i] = x[i] * a.scale;
        kn[i] = kx[i];
      }
    }
    uint4 qh, ql;
    split2(qv[0], qv[1], qh.x, ql.x);
    split2(qv[2], qv[3], qh.y, ql.y);
    split2(qv[4], qv[5], qh.z, ql.z);
    split2(qv[6], qv[7], qh.w, ql.w);
    lds_q[0][w][lane] = qh;                                      // hi, lo planes of the query operand, for every wave
    lds_q[1][w][lane] = ql;
    if (l16 == 0) {                                              // the new key: into LDS for the row's last block, and into the cache
      const u32x4 knew = {pk_bf16(kn[0], kn[1]), pk_bf16(kn[2], kn[3]), pk_bf16(kn[4], kn[5]), pk_bf16(kn[6], kn[7])};
      *reinterpret_cast<u32x4*>(lds_kn + d0) = knew;
      if (blockIdx.z == 0) *reinterpret_cast<u32x4*>(Kc + (size_t)slot * DH + d0) = knew;
    }
  }
  if (w == VW) {                                                 // the new value likewise
#pragma unroll
    for (int i = 0; i < DH / 64; ++i) {
      const bf16_t h = (bf16_t)pk_bf16(vraw[i], 0.f);
      lds_vn[i * 64 + lane] = h;
      if (blockIdx.z == 0) Vc[vt_index(slot, i * 64 + lane, DH)] = h;
    }
  }
  lds_barrier();                                                 // the query operand and the new key are in LDS for every wave
  f32x4 O[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) O[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m_run[NV], l_run[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) { m_run[v] = NEG; l_run[v] = 0.f; }
  float* myp = lds_p[w];
  auto step = [&](Blk& Bk, int kb) {
    if (kb + 31 >= slot) {                                       // (scalar) the row's last block or beyond: patch the new key in
#pragma unroll
      for (int tile = 0; tile < 2; ++tile)
        if (kb + tile * 16 + l16 == slot) {
#pragma unroll
          for (int t = 0; t < T; ++t) Bk.k[tile][t] = *reinterpret_cast<const u32x4*>(lds_kn + t * 32 + lq * 8);
        }
    }
    f32x4 sc[2];
#pragma unroll
    for (int tile = 0; tile < 2; ++tile) {
      sc[tile] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const u32x4 kk = Bk.k[tile][t];
        const uint4 kf = make_uint4(kk.x, kk.y, kk.z, kk.w);
        sc[tile] = mfma_bf16(lds_q[0][t][lane], kf, sc[tile]);
        sc[tile] = mfma_bf16(lds_q[1][t][lane], kf, sc[tile]);
      }
    }
    // accumulator register v of lane (lq, l16) is head lq * NV + v (beyond G: the last head again), key kb + tile * 16 + l16
    const bool ok0 = kb + l16 <= slot, ok1 = kb + 16 + l16 <= slot;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const float mx = group_max16(fmaxf(ok0 ? sc[0][v] : NEG, ok1 ? sc[1][v] : NEG));
      const float mn = fmaxf(m_run[v], mx);
      const float corr = __expf(m_run[v] - mn);
      const float p0 = ok0 ? __expf(sc[0][v] - mn) : 0.f, p1 = ok1 ? __expf(sc[1][v] - mn) : 0.f;
      l_run[v] = l_run[v] * corr + group_sum<16>(p0 + p1);
      m_run[v] = mn;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) O[ct][v] *= corr;
      myp[(lq * NV + v) * PS + l16] = p0;
      myp[(lq * NV + v) * PS + 16 + l16] = p1;
    }
    __builtin_amdgcn_wave_barrier();                             // LDS operations of one wave complete in order
    uint4 ph, pl;                                                // P in operand layout: row l16's head, keys lq * 8 .. + 8
    {
      const float* pr = myp + ((l16 >> 2) * NV + min(l16 & 3, NV - 1)) * PS + lq * 8;
      const float4 u = *reinterpret_cast<const float4*>(pr), x = *reinterpret_cast<const float4*>(pr + 4);
      split2(u.x, u.y, ph.x, pl.x);
      split2(u.z, u.w, ph.y, pl.y);
      split2(x.x, x.y, ph.z, pl.z);
      split2(x.z, x.w, ph.w, pl.w);
    }
    __builtin_amdgcn_wave_barrier();
    if (kb + 31 >= slot) {                                       // (scalar) new value in, keys beyond the row's last one out
      const int at = slot - kb - lq * 8;                         // where slot lies among this lane's 8 keys
      unsigned keep[4], own[4], vnew[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) vnew[ct] = lds_vn[ct * 16 + l16] * 0x10001u;
      vt_first(at, keep);
#pragma unroll
      for (int e = 0; e < 4; ++e) own[e] = at == 2 * e ? 0xffffu : at == 2 * e + 1 ? 0xffff0000u : 0u;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) Bk.v[ct][e] = (Bk.v[ct][e] & keep[e]) | (vnew[ct] & own[e]);
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const uint4 vf = make_uint4(Bk.v[ct].x, Bk.v[ct].y, Bk.v[ct].z, Bk.v[ct].w);
      O[ct] = mfma_bf16(ph, vf, O[ct]);
      O[ct] = mfma_bf16(pl, vf, O[ct]);
    }
  };
  if (DH == 64 && n_steps == 1) step(A, wz * 32);                // (scalar) no second block to request (a third copy spills at 128)
  else for (int i = 0; i < n_steps; i += 2) {
    const int kb = (i * NZ + wz) * 32;
    fetch(B, kb + 32 * NZ);
    __builtin_amdgcn_sched_barrier(0);
    step(A, kb);
    __builtin_amdgcn_sched_barrier(0);
    if (i + 1 < n_steps) {                                       // (scalar condition)
      fetch(A, kb + 64 * NZ);
      __builtin_amdgcn_sched_barrier(0);
      step(B, kb + 32 * NZ);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // merge the waves: head lq * NV + v lives in the lanes of DPP row lq
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int g = lq * NV + v;
    if (g < G) {
      if (l16 == 0) { s_ml[w][g][0] = m_run[v]; s_ml[w][g][1] = l_run[v]; }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) s_o[w][g][ct * 16 + l16] = O[ct][v];
    }
  }
  lds_barrier();
  bf16_t* __restrict__ ao = (bf16_t*)a.ao;
  for (int idx = tid; idx < G * DH; idx += NW * 64) {
    const int g = idx / DH, i = idx % DH;
    float mn = NEG;
#pragma unroll
    for (int q = 0; q < NW; ++q) mn = fmaxf(mn, s_ml[q][g][0]);
    float den = 0.f, num = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const float c = __expf(s_ml[q][g][0] - mn);
      den += c * s_ml[q][g][1];
      num += c * s_o[q][g][i];
    }
    if (extra_ > 1) {                                            // (uniform)
      float* __restrict__ o = a.split + ((((size_t)r * a.KVH + kvh) * extra_ + blockIdx.z) * G + g) * (DH + 2);
      o[i] = num;
      if (i == 0) { o[DH] = mn; o[DH + 1] = den; }
    } else {
      act_store<bf16_t>(ao, r, kvh * G * DH + idx, a.ao_K, num / den);
    }
  }
}

// One workgroup per (query head, row): the n <= 8 partial results of k_attn_dec_bf16, in their order.
template <int DH>
__global__ __launch_bounds__(DH) void k_attn_merge(AttnArgs a, int n) {
  const int h = blockIdx.x, r = blockIdx.y, G = a.G, kvh = h / G, g = h % G, i = threadIdx.x;
  const float* __restrict__ p = a.split + (((size_t)r * a.KVH + kvh) * n * G + g) * (DH + 2);
  float m[8], l[8], o[8];
#pragma unroll
  for (int z = 0; z < 8; ++z) {                                  // (requested together; beyond n: the last one again, dropped)
    const float* q = p + (size_t)min(z, n - 1) * G * (DH + 2);
    m[z] = q[DH]; l[z] = q[DH + 1]; o[z] = q[i];
  }
  if (r >= *a.rd.n_rows) return;
  float mn = -1e30f, den = 0.f, num = 0.f;
#pragma unroll
  for (int z = 0; z < 8; ++z) mn = fmaxf(mn, m[z]);
#pragma unroll
  for (int z = 0; z < 8; ++z) {
    const float c = z < n ? __expf(m[z] - mn) : 0.f;
    den += c * l[z];
    num += z < n ? c * o[z] : 0.f;
  }
  act_store<bf16_t>((bf16_t*)a.ao, r, h * DH + i, a.ao_K, num / den);
}

// Append-only launch of a multi-entry pass: rotate the new key, round key and value to bf16 and write them to the
// entry's cache slot - what k_attn_dec_bf16 does in its prologue, without the attention around it.  One wave per
// (8 entries, KV head).  The value cache keeps 8 consecutive slots of a column in 16 bytes (vt_index): where 8 entries in a row
// are such a block of slots of one batch row - all but the ends of a prefill run - the wave in whose window the block begins
// gathers a column's 8 values from the 8 rows per lane and stores 16 bytes; the other entries of the window go 2 bytes per
// entry and column, as in the attention kernel.  (One entry per wave with 2-byte stores: 125 us for 4096 entries x 32 heads
// x 128 columns, now 49, of which 30 are its 192 MB at the rate of a copy.)
template <int DH>
__global__ __launch_bounds__(64) void k_kv_append_bf16(AttnArgs a) {
  constexpr int LPK = DH / 8, KEYS = 64 / LPK;                   // lanes per key, keys per wave and round
  const int n_rows = *a.rd.n_rows, r0 = blockIdx.y * 8;
  if (r0 >= n_rows) return;
  const int lane = threadIdx.x, kvh = blockIdx.x, S = a.max_seq, n_here = min(8, n_rows - r0);
  // lane i: the descriptor of entry r0 - 7 + i, so that lanes 7 .. 14 hold the window and its blocks lie in lanes 0 .. 21
  const int ri = r0 - 7 + lane;
  const bool listed = lane < 22 && ri >= 0 && ri < n_rows;
  const int at = min(max(ri, 0), n_rows - 1), e_b = a.rd.b[at], e_slot = a.rd.slot[at];
  const size_t head = (size_t)S * DH;
  bf16_t* __restrict__ kc = (bf16_t*)a.kcache + a.layer_off;
  bf16_t* __restrict__ vc = (bf16_t*)a.vcache + a.layer_off;
  // ---- keys: 8 elements per lane
  const int chunk = lane % LPK, pchunk = chunk ^ (LPK / 2);
  const bool upper = chunk >= LPK / 2;
#pragma unroll
  for (int k0 = 0; k0 < 8; k0 += KEYS) {
    const int e = k0 + lane / LPK, r = r0 + min(e, n_here - 1);
    const float* __restrict__ y = a.y + (size_t)r * a.dqkv + (size_t)(a.H + kvh) * DH;
    const float* __restrict__ cs = a.rope + (size_t)r * DH + 2 * (chunk % (LPK / 2)) * 8;
    float x[8], xp[8], c16[16];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float4 u = reinterpret_cast<const float4*>(y + chunk * 8)[i], w = reinterpret_cast<const float4*>(y + pchunk * 8)[i];
      x[4 * i] = u.x; x[4 * i + 1] = u.y; x[4 * i + 2] = u.z; x[4 * i + 3] = u.w;
      xp[4 * i] = w.x; xp[4 * i + 1] = w.y; xp[4 * i + 2] = w.z; xp[4 * i + 3] = w.w;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 u = reinterpret_cast<const float4*>(cs)[i];
      c16[4 * i] = u.x; c16[4 * i + 1] = u.y; c16[4 * i + 2] = u.z; c16[4 * i + 3] = u.w;
    }
    unsigned pk[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v2[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int q = 2 * i + j;
        const float c = a.use_rope ? c16[2 * q] : 1.f, sn = a.use_rope ? c16[2 * q + 1] : 0.f;
        v2[j] = upper ? x[q] * c + xp[q] * sn : x[q] * c - xp[q] * sn;
      }
      pk[i] = pk_bf16(v2[0], v2[1]);
    }
    const int b = __shfl(e_b, 7 + e), slot = __shfl(e_slot, 7 + e);
    if (e < n_here)
      *reinterpret_cast<uint4*>(kc + ((size_t)b * a.KVH + kvh) * head + (size_t)slot * DH + chunk * 8) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
  }
  // ---- values.  follows: bit i = entry i is the next position of entry i - 1; 7 of them after a slot that is a multiple of 8
  // make a block
  const int b_prev = __shfl_up(e_b, 1), slot_prev = __shfl_up(e_slot, 1);
  const u64 follows = __ballot(lane > 0 && listed && ri > 0 && e_b == b_prev && e_slot == slot_prev + 1);
  const int first = lane - (e_slot & 7);                         // lane of the block's first entry
  const bool in_window = listed && lane >= 7 && lane < 15;
  const bool full = in_window && ((follows >> (first + 1)) & 0x7f) == 0x7f;
  const u64 starts = __ballot(full && (e_slot & 7) == 0);        // at most one bit
  const u64 single = __ballot(in_window && !full);
  const float* __restrict__ yv = a.y + (size_t)(a.H + a.KVH + kvh) * DH;
  if (starts) {
    const int f = __builtin_ctzll(starts), b = __builtin_amdgcn_readlane(e_b, f), slot = __builtin_amdgcn_readlane(e_slot, f);
#pragma unroll
    for (int c0 = 0; c0 < DH; c0 += 64) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = yv[(size_t)(r0 - 7 + f + e) * a.dqkv + c0 + lane];
      unsigned pk[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) pk[i] = pk_bf16(x[2 * i], x[2 * i + 1]);
      *reinterpret_cast<uint4*>(vc + ((size_t)b * a.KVH + kvh) * head + vt_index(slot, c0 + lane, DH)) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    }
  }
  if (single) {                                                  // all of the window's values requested together
    float x[8][DH / 64];
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int c = 0; c < DH / 64; ++c) x[e][c] = yv[(size_t)(r0 + min(e, n_here - 1)) * a.dqkv + c * 64 + lane];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if ((single >> (7 + e)) & 1) {                             // (scalar)
        const int b = __builtin_amdgcn_readlane(e_b, 7 + e), slot = __builtin_amdgcn_readlane(e_slot, 7 + e);
#pragma unroll
        for (int c = 0; c < DH / 64; ++c)
          vc[((size_t)b * a.KVH + kvh) * head + vt_index(slot, c * 64 + lane, DH)] = f2bf(x[e][c]);
      }
  }
}

// Maximum / sum over the four lanes that share lane % 16 (lanes 16 apart), in all of them: two lane swaps on the vector ALU.
__device__ __forceinline__ float quarter_max(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quarter_sum(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The queries of one wave of the two kernels below, rotated and scaled (in base-2 units), to LDS in operand layout [set][32 columns]
// [hi, lo][lane]: 16 entries from `first` on (beyond the last row: that one again) of heads h0 and h0 + 1 (PAIR), or 32 entries of head
// h0.  The lanes go along the rows, 4 columns each (16 rows x 16 pieces of 32 bytes at once took the memory pipeline 4 times as
// long).  All of a set's loads (PAIR: both sets') are requested together: left to the compiler they went out four at a time, 16 trips to
// memory one after the other, 20 us of a wave's life.
template <int DH, bool PAIR>
__device__ __forceinline__ void queries_to_lds(const AttnArgs& a, int first, int n_rows, int h0, uint4 (*q)[DH / 32][2][64]) {
  constexpr int LPR = DH / 4, RPI = 64 / LPR, NI = 16 / RPI, SETS = PAIR ? 2 : 1;   // lanes per row, rows per instruction, instructions
  const int lane = threadIdx.x & 63, c4 = (lane % LPR) * 4, sub = lane / LPR;
  const float scale = a.scale * 1.4426950408889634f, sg = c4 >= DH / 2 ? 1.f : -1.f;
#pragma unroll
  for (int s0 = 0; s0 < 2; s0 += SETS) {
    float4 x[SETS][NI];
    auto row = [&](int i) { return min(first + (PAIR ? 0 : 16 * s0) + i * RPI + sub, n_rows - 1); };
    auto load = [&](float4 (&v)[SETS][NI], int col) {
#pragma unroll
      for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int i = 0; i < NI; ++i) v[s][i] = *reinterpret_cast<const float4*>(a.y + (size_t)row(i) * a.dqkv + (size_t)(h0 + s) * DH + col);
    };
    load(x, c4);
    if (a.use_rope) {                                            // (uniform)
      float4 xp[SETS][NI], c[NI], d[NI];                         // cos, sin, cos, sin
      load(xp, c4 ^ (DH / 2));
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float4* __restrict__ cs = reinterpret_cast<const float4*>(a.rope + (size_t)row(i) * DH + 2 * (c4 % (DH / 2)));
        c[i] = cs[0]; d[i] = cs[1];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < SETS; ++s)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float4& v = x[s][i];
          const float4 w = xp[s][i];
          v.x = v.x * c[i].x + sg * (w.x * c[i].y); v.y = v.y * c[i].z + sg * (w.y * c[i].w);
          v.z = v.z * d[i].x + sg * (w.z * d[i].y); v.w = v.w * d[i].z + sg * (w.w * d[i].w);
        }
    }
#pragma unroll
    for (int s = 0; s < SETS; ++s)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        uint2 qh, ql;
        split2(x[s][i].x * scale, x[s][i].y * scale, qh.x, ql.x);
        split2(x[s][i].z * scale, x[s][i].w * scale, qh.y, ql.y);
        const int at = ((c4 & 31) >> 3) * 16 + i * RPI + sub;    // operand lane of the row, columns c4 & ~7 .. + 7
        *reinterpret_cast<uint2*>((char*)&q[s0 + s][c4 >> 5][0][at] + (c4 & 4) * 2) = qh;
        *reinterpret_cast<uint2*>((char*)&q[s0 + s][c4 >> 5][1][at] + (c4 & 4) * 2) = ql;
      }
    __builtin_amdgcn_sched_barrier(0);                           // one set's loads at a time (registers)
  }
  __builtin_amdgcn_wave_barrier();                               // (a wave's LDS operations complete in order)
}

// Causal attention on the matrix cores for a multi-entry pass whose entries come in runs of consecutive positions of
// one batch row (prefill); every key and value of the pass is already cached (the append-only launch ran before).
// One wave takes two sets of 16 queries that read the same keys: two heads of one KV head over 16 entries (PAIR), or one
// head over 32 entries, so that a key or value fragment fetched from L2 feeds four products.  Per block of 32 keys:
//   S^T = K Q^T: a lane holds the scores of ONE query (lane % 16) against 8 keys, so the softmax statistics are one value per
//     lane, reduced in the lane and over the four lanes of the query (sums only at the end).  Row i of key tile t is key
//     8 (i / 4) + 4 t + i % 4: the 8 keys a lane ends up with are 8 (lane / 16) .. + 7, which is the operand layout of P.
//   O^T += V^T P^T with P straight from those registers (hi + lo bf16, as Q: both enter at float32 precision); V^T tiles
//     straight from the cache, keys beyond the run's last one zeroed (0 x NaN is NaN).  The accumulator holds four
//     consecutive columns of one query per lane: 8-byte stores.
// The keys of the next block are requested when this block's have been used, and the values likewise.
// Per launch at 4096 entries: 32 heads x 128 columns, prompts of 64 - 512: 80 us, with the queries' loads requested together 74; 32 heads
// over 8 KV heads, 512: 90 -> 81; contexts up to 2000: 176 -> 164.  What bounds it now, by a fit over those: 1.5 us per block of 32 keys
// and pair of waves of a SIMD, of which the matrix instructions are 1, and about 15 us of a wave's life outside its blocks.
// What bounded the version before (16 queries of one head per wave, the query along the registers, P through LDS, 366 registers) was not arithmetic either: one descriptor read after the
// other, and barriers that waited for the prefetched block every time.
template <int DH, bool PAIR>
__global__ __launch_bounds__(64, 2) void k_attn_mfma_bf16(AttnArgs a) {
  constexpr int T = DH / 32, CT = DH / 16, E = PAIR ? 16 : 32;
  constexpr float NEG = -1e30f;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __shared__ uint4 lds_q[2][T][2][64];                           // (in registers the queries spill at 128 columns)
  const int n_rows = *a.rd.n_rows, r0 = (gridDim.y - 1 - blockIdx.y) * E;   // the longest contexts first
  if (r0 >= n_rows) return;
  const int lane = threadIdx.x, l16 = lane & 15, lq = lane >> 4, S = a.max_seq, G = a.G;
  const int h0 = PAIR ? 2 * blockIdx.x : blockIdx.x, kvh = h0 / G;
  const int n_here = min(E, n_rows - r0), mine = r0 + min(lane, n_here - 1);
  const int e_b = a.rd.b[mine], e_slot = a.rd.slot[mine];        // lane e: entry e's batch row and position in the cache
  const int b_prev = __shfl_up(e_b, 1);                          // (by all lanes: an inactive one would read as 0)
  u64 starts = __ballot(lane < n_here && (lane == 0 || e_b != b_prev));
  queries_to_lds<DH, PAIR>(a, r0, n_rows, h0, lds_q);
  while (starts) {
    const int s0 = __builtin_ctzll(starts);
    starts &= starts - 1;
    const int s1 = starts ? __builtin_ctzll(starts) : n_here;    // entries s0 .. s1 - 1 belong to batch row b, positions ascend
    const int b = __builtin_amdgcn_readlane(e_b, s0), max_slot = __builtin_amdgcn_readlane(e_slot, s1 - 1);
    const bf16_t* __restrict__ Kc = (const bf16_t*)a.kcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH;
    const bf16_t* __restrict__ Vc = (const bf16_t*)a.vcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH;
    u32x4 K[2][T], V[CT];
    const int key_lane = (l16 >> 2) * 8 + (l16 & 3);
    auto fetch_k = [&](int kb) {                                 // (keys beyond the run's last one: that one again, masked)
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        const bf16_t* kr = Kc + (size_t)min(kb + key_lane + t2 * 4, max_slot) * DH + lq * 8;
#pragma unroll
        for (int t = 0; t < T; ++t) K[t2][t] = *reinterpret_cast<const u32x4*>(kr + t * 32);
      }
    };
    auto fetch_v = [&](int kb) {
      const bf16_t* vb = Vc + (size_t)(min(kb, max_slot & ~31) >> 5) * (32 * DH) + lane * 8;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) V[ct] = *reinterpret_cast<const u32x4*>(vb + ct * 512);
    };
    fetch_k(0);
    fetch_v(0);
    int slot[2];                                                 // a query's position; -1: not of this run, every key masked
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int e = l16 + (PAIR ? 0 : 16 * s), sl = __shfl(e_slot, e);
      slot[s] = (e >= s0 && e < s1) ? sl : -1;
    }
    f32x4 O[2][CT];
    float m_run[2] = {NEG, NEG}, l_run[2] = {0.f, 0.f};          // (l_run: this lane's keys only)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) O[s][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int kb = 0; kb <= max_slot; kb += 32) {
      f32x4 sc[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s) sc[s][0] = sc[s][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)                           // (four independent chains)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const uint4 q = lds_q[s][t][hl][lane];
            sc[s][0] = mfma_bf16(__builtin_bit_cast(uint4, K[0][t]), q, sc[s][0]);
            sc[s][1] = mfma_bf16(__builtin_bit_cast(uint4, K[1][t]), q, sc[s][1]);
          }
      __builtin_amdgcn_sched_barrier(0);
      fetch_k(kb + 32);
      __builtin_amdgcn_sched_barrier(0);
      uint4 ph[2], pl[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int left = slot[s] - kb - lq * 8;                  // keys 0 .. left of this lane's 8 are valid
        float x[8], mx = NEG;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          x[e] = e <= left ? sc[s][e >> 2][e & 3] : NEG;
          mx = fmaxf(mx, x[e]);
        }
        const float mn = fmaxf(m_run[s], quarter_max(mx));
        if (__any(mn > m_run[s])) {                              // (uniform) the running maximum of some query moves
          const float corr = __builtin_amdgcn_exp2f(m_run[s] - mn);
          l_run[s] *= corr;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) O[s][ct] *= corr;
          m_run[s] = mn;
        }
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = e <= left ? __builtin_amdgcn_exp2f(x[e] - mn) : 0.f;
        l_run[s] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        split2(p[0], p[1], ph[s].x, pl[s].x);
        split2(p[2], p[3], ph[s].y, pl[s].y);
        split2(p[4], p[5], ph[s].z, pl[s].z);
        split2(p[6], p[7], ph[s].w, pl[s].w);
      }
      if (kb + 31 > max_slot) {                                  // (scalar) zero the values of keys beyond the run's last one
        unsigned keep[4];
        vt_first(max_slot + 1 - kb - lq * 8, keep);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int e = 0; e < 4; ++e) V[ct][e] &= keep[e];
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const uint4 vf = __builtin_bit_cast(uint4, V[ct]);
        O[0][ct] = mfma_bf16(vf, ph[0], O[0][ct]);
        O[1][ct] = mfma_bf16(vf, ph[1], O[1][ct]);
        O[0][ct] = mfma_bf16(vf, pl[0], O[0][ct]);
        O[1][ct] = mfma_bf16(vf, pl[1], O[1][ct]);
      }
      __builtin_amdgcn_sched_barrier(0);
      fetch_v(kb + 32);
      __builtin_amdgcn_sched_barrier(0);
    }
    bf16_t* __restrict__ ao = (bf16_t*)a.ao;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const float inv = 1.0f / quarter_sum(l_run[s]);
      if (slot[s] < 0) continue;
      const int m = r0 + l16 + (PAIR ? 0 : 16 * s);
      bf16_t* __restrict__ dst = ao + act_idx<bf16_t>(m, (h0 + (PAIR ? s : 0)) * DH + lq * 4, a.ao_K);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {                          // 16 columns on: half an operand tile (256 elements)
        const f32x4 o = O[s][ct] * inv;
        *reinterpret_cast<uint2*>(dst + ct * 256) = make_uint2(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]));
      }
    }
  }
}

// 16 bytes per lane from memory to LDS at `lds` + 16 x lane.  In asm, because the compiler puts a wait for every such load of its builtin
// in front of this kernel's next read of LDS; the kernel's own waits count them.
__device__ __forceinline__ void lds_load16(const bf16_t* src, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory", "m0");
}

// The same with the keys and values of a KV head shared by the four waves of a workgroup: a wave takes two heads over 16 entries as
// above, the four of them the head pairs of the KV head, times as many groups of 16 entries as that leaves waves for (2, 4, 8 heads per
// KV head: 64, 32, 16 entries).  Blocks of 32 keys go to LDS in operand order (a ring of S stages, global_load_lds: no registers, one
// quarter of a block per wave), so the register room goes to the queries, which are read from LDS once instead of per block, and a
// key or value crosses from L2 to a compute unit a quarter as often.  The same bits as above.  What bounds it, by the same fit: 1.2 us per
// block and pair of waves, vector next to matrix instructions; the 15 us outside are the same.
// us per launch at 4096 entries, 32 heads of 128 columns over 8: prompts of 512 81 -> 73, contexts up to 2000 164 -> 136.
template <int DH>
__global__ __launch_bounds__(256, 2) void k_attn_mfma_shared_bf16(AttnArgs a) {
  constexpr int T = DH / 32, CT = DH / 16, S = 4, F = 2 * T + CT;   // F fragments per block; waves 0, 1: keys, 2, 3: values, T each
  constexpr float NEG = -1e30f;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __shared__ u32x4 ring[S][F][64];
  static_assert(S * F == 4 * 2 * T * 2, "the four waves' queries pass through the ring");
  const int n_rows = *a.rd.n_rows, G = a.G, pairs = G >> 1, E = 64 / pairs;
  const int r0 = (gridDim.y - 1 - blockIdx.y) * E;               // the longest contexts first
  if (r0 >= n_rows) return;
  const int lane = threadIdx.x & 63, w = wave_index(), l16 = lane & 15, lq = lane >> 4, max_seq = a.max_seq;
  const int kvh = blockIdx.x, h0 = kvh * G + 2 * (w % pairs), e0 = 16 * (w / pairs);
  const int n_here = min(E, n_rows - r0), mine = r0 + min(lane, n_here - 1);
  const int e_b = a.rd.b[mine], e_slot = a.rd.slot[mine];        // lane e: entry e's batch row and position in the cache
  const int b_prev = __shfl_up(e_b, 1);                          // (by all lanes: an inactive one would read as 0)
  u64 starts = __ballot(lane < n_here && (lane == 0 || e_b != b_prev));
  uint4(*q_lds)[T][2][64] = reinterpret_cast<uint4(*)[T][2][64]>(&ring[0][0][0] + w * (2 * T * 2 * 64));
  queries_to_lds<DH, true>(a, r0 + e0, n_rows, h0, q_lds);       // (through the wave's quarter of the ring)
  uint4 Q[2][T][2];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int hl = 0; hl < 2; ++hl) Q[s][t][hl] = q_lds[s][t][hl][lane];
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wave has its queries: the ring is free
  while (starts) {                                               // (the same for the four waves, as are s0, s1 and n_blk)
    const int s0 = __builtin_ctzll(starts);
    starts &= starts - 1;
    const int s1 = starts ? __builtin_ctzll(starts) : n_here;    // entries s0 .. s1 - 1 belong to batch row b, positions ascend
    const int b = __builtin_amdgcn_readlane(e_b, s0), max_slot = __builtin_amdgcn_readlane(e_slot, s1 - 1), n_blk = (max_slot >> 5) + 1;
    const int q0 = max(s0, e0), q1 = min(s1, e0 + 16);           // this wave's entries of the run (none: it only loads)
    const int my_min = q0 < q1 ? __builtin_amdgcn_readlane(e_slot, q0) : 0, my_max = q0 < q1 ? __builtin_amdgcn_readlane(e_slot, q1 - 1) : -1;
    const size_t head = ((size_t)b * a.KVH + kvh) * (size_t)max_seq * DH;
    const bf16_t* __restrict__ Kc = (const bf16_t*)a.kcache + a.layer_off + head;
    const bf16_t* __restrict__ Vc = (const bf16_t*)a.vcache + a.layer_off + head;
    const int e_mine = e0 + l16, sl = __shfl(e_slot, e_mine);
    const int slot = (e_mine >= q0 && e_mine < q1) ? sl : -1;    // the lane's query's position; -1: not of this run, never stored
    // Row i of key tile t2 is key 8 (i / 4) + 4 t2 + i % 4; keys beyond the run's last one: that one again, masked.  Blocks beyond
    // the last one: it again, never read.
    const int key_lane = (l16 >> 2) * 8 + (l16 & 3) + (w & 1) * 4;
    auto issue = [&](int i) {
      const int kb = min(i, n_blk - 1) * 32;
      const bf16_t* src = w < 2 ? Kc + (size_t)min(kb + key_lane, max_slot) * DH + lq * 8 : Vc + (size_t)kb * DH + (w - 2) * (T * 512) + lane * 8;
      const int step = w < 2 ? 32 : 512;                         // (scalar)
      const unsigned dst = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)&ring[i % S][w * T][0];
#pragma unroll
      for (int j = 0; j < T; ++j) lds_load16(src + j * step, __builtin_amdgcn_readfirstlane(dst + j * 1024));
    };
    f32x4 O[2][CT];
    float m_run[2] = {NEG, NEG}, l_run[2] = {0.f, 0.f};          // (l_run: this lane's keys only)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) O[s][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < S - 1; ++i) issue(i);
    for (int i = 0; i < n_blk; ++i) {
      // this wave's part of block i has landed, its reads of block i - 1 are back; then the same of every wave
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((S - 2) * T) : "memory");
      issue(i + S - 1);
      const int kb = i * 32;
      if (kb > my_max) continue;                                 // (scalar) nothing here that an entry of this wave sees
      const u32x4(*blk)[64] = ring[i % S];
      f32x4 sc[2][2];
#pragma unroll
      for (int s = 0; s < 2; ++s) sc[s][0] = sc[s][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const uint4 k0 = __builtin_bit_cast(uint4, blk[t][lane]), k1 = __builtin_bit_cast(uint4, blk[T + t][lane]);
#pragma unroll
        for (int hl = 0; hl < 2; ++hl)                           // (four independent chains)
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const uint4 q = Q[s][t][hl];
            sc[s][0] = mfma_bf16(k0, q, sc[s][0]);
            sc[s][1] = mfma_bf16(k1, q, sc[s][1]);
          }
      }
      u32x4 V[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) V[ct] = blk[2 * T + ct][lane];
      const bool edge = kb + 31 > my_min;                        // (scalar) some entry of the run does not see the whole block
      const int left = slot - kb - lq * 8;                       // keys 0 .. left of this lane's 8 are valid
      uint4 ph[2], pl[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        float x[8], mx = NEG;
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = sc[s][e >> 2][e & 3];
        if (edge) {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = e <= left ? x[e] : NEG;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, x[e]);
        const float mn = fmaxf(m_run[s], quarter_max(mx));
        if (__any(mn > m_run[s])) {                              // (uniform) the running maximum of some query moves
          const float corr = __builtin_amdgcn_exp2f(m_run[s] - mn);
          l_run[s] *= corr;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) O[s][ct] *= corr;
          m_run[s] = mn;
        }
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(x[e] - mn);
        if (edge) {
#pragma unroll
          for (int e = 0; e < 8; ++e) p[e] = e <= left ? p[e] : 0.f;
        }
        l_run[s] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        split2(p[0], p[1], ph[s].x, pl[s].x);
        split2(p[2], p[3], ph[s].y, pl[s].y);
        split2(p[4], p[5], ph[s].z, pl[s].z);
        split2(p[6], p[7], ph[s].w, pl[s].w);
      }
      if (kb + 31 > my_max) {                                    // (scalar) zero the values of keys beyond the wave's last one
        unsigned keep[4];
        vt_first(my_max + 1 - kb - lq * 8, keep);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int e = 0; e < 4; ++e) V[ct][e] &= keep[e];
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const uint4 vf = __builtin_bit_cast(uint4, V[ct]);
        O[0][ct] = mfma_bf16(vf, ph[0], O[0][ct]);
        O[1][ct] = mfma_bf16(vf, ph[1], O[1][ct]);
        O[0][ct] = mfma_bf16(vf, pl[0], O[0][ct]);
        O[1][ct] = mfma_bf16(vf, pl[1], O[1][ct]);
      }
    }
    // The clamped loads of the last stages still write to LDS; then the ring is free for the next run.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    bf16_t* __restrict__ ao = (bf16_t*)a.ao;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const float inv = 1.0f / quarter_sum(l_run[s]);
      if (slot < 0) continue;
      bf16_t* __restrict__ dst = ao + act_idx<bf16_t>(r0 + e_mine, (h0 + s) * DH + lq * 4, a.ao_K);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {                          // 16 columns on: half an operand tile (256 elements)
        const f32x4 o = O[s][ct] * inv;
        *reinterpret_cast<uint2*>(dst + ct * 256) = make_uint2(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]));
      }
    }
  }
}

// The same for a multi-entry pass whose runs are short (speculative windows, full-prefix work lists): up to 16 / G consecutive
// entries of a row, times the G query heads of the KV head, are the 16 queries of one pass over the row's keys, shared by NW
// waves: wave w takes the 32-key blocks w, w + NW, ..., and the waves' partial results are merged through LDS.  A workgroup
// whose entry is not the first of its group (the run's first entry, or a position that is a multiple of 16 / G) has nothing to
// do.  A value that is not finite must not reach earlier entries of its group (0 x NaN is NaN): the blocks with the group's own
// keys are looked through for one; entries that see it get NaN, the products of the others take zeros.  (80 entries in 16 windows of 5,
// 25 heads of 64, 110 keys: 22.0 us with a pass per entry, 9.9 so; 16 entries of one each: 8.5 and 5.9.  With the queries requested ahead of
// the descriptors, 150 keys: 26 entries of 12 heads 6.2 -> 5.9, 12 of 25 7.15 -> 6.85, 80 of 25 9.9 -> 9.7, 160 of 32 x 128 37.1 -> 35.6.)
template <int DH, int NW, bool ROPE>
__global__ __launch_bounds__(NW * 64, 2) void k_attn_runs_bf16(ATTN_ARGS) {   // extra: entries
  const AttnArgs a = attn_args<DH>(y_, b_, slot_, kcache_, vcache_, H_, KVH_, S_, extra_, n_rows_, ao_, rope_, nullptr);
  constexpr int T = DH / 32, CT = DH / 16;
  constexpr float NEG = -1e30f;
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __shared__ u32x4 lds_q[T][2][64];                              // [32 columns][hi, lo][lane]
  __shared__ float s_ml[NW][16][2];
  __shared__ __attribute__((aligned(16))) float s_o[NW][16][DH + 4];
  const int n_rows = *a.rd.n_rows, r = blockIdx.y, kvh = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), l16 = lane & 15, lq = lane >> 4, S = a.max_seq;
  const int G = H_ / KVH_, lg = __builtin_ctz(G), M = 16 >> lg;
  // lane i: entry r - 1 + i; the group is entry r and those that continue it up to the next multiple of M.  The descriptors and the
  // queries of all M entries that may be in it are requested together, before the row count is known (the buffers hold every row
  // the grid covers); what belongs to no entry of the group is masked below.
  const int ri = r - 1 + lane, r_last = extra_ - 1;
  const int at = min(max(ri, 0), r_last), e_b = a.rd.b[at], e_slot = a.rd.slot[at];
  constexpr int LPR = DH / 4, RPI = 64 / LPR, QI = (16 / RPI + NW - 1) / NW;   // lanes per query, queries per instruction, instructions per wave
  const int c4 = (lane % LPR) * 4;
  float4 qx[QI], qp[QI], qc[QI][2];
#pragma unroll
  for (int i = 0; i < QI; ++i) {
    const int col = min((i * NW + w) * RPI + lane / LPR, 15), re = min(r + (col >> lg), r_last);
    const float* __restrict__ y = a.y + (size_t)re * a.dqkv + (size_t)(kvh * G + (col & (G - 1))) * DH;
    qx[i] = *reinterpret_cast<const float4*>(y + c4);
    if (ROPE) {
      const float4* __restrict__ cs = reinterpret_cast<const float4*>(a.rope + (size_t)re * DH + 2 * (c4 % (DH / 2)));
      qp[i] = *reinterpret_cast<const float4*>(y + (c4 ^ (DH / 2)));
      qc[i][0] = cs[0]; qc[i][1] = cs[1];                        // cos, sin, cos, sin
    }
  }
  if (r >= n_rows) return;
  const bool listed = ri >= 0 && ri < n_rows;
  const int b = __builtin_amdgcn_readlane(e_b, 1), slot0 = __builtin_amdgcn_readlane(e_slot, 1);
  const u64 follows = __ballot(listed && e_b == b && e_slot == slot0 + lane - 1);
  if ((follows & 1) && (slot0 & (M - 1)) != 0) return;           // (uniform) entry r - 1's group holds this entry
  const u64 group = __ballot(lane >= 2 && lane <= M && (e_slot & (M - 1)) != 0) & follows;
  const int n = 1 + __builtin_ctzll(~(group >> 2)), n_col = n << lg, max_slot = slot0 + n - 1;
  const bf16_t* __restrict__ Kc = (const bf16_t*)a.kcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH;
  const bf16_t* __restrict__ Vc = (const bf16_t*)a.vcache + a.layer_off + ((size_t)b * a.KVH + kvh) * (size_t)S * DH;
  u32x4 K[2][T], V[CT];
  const int key_lane = (l16 >> 2) * 8 + (l16 & 3);               // (key order as in k_attn_mfma_bf16)
  auto fetch_k = [&](int kb) {
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
      const bf16_t* kr = Kc + (size_t)min(kb + key_lane + t2 * 4, max_slot) * DH + lq * 8;
#pragma unroll
      for (int t = 0; t < T; ++t) K[t2][t] = *reinterpret_cast<const u32x4*>(kr + t * 32);
    }
  };
  auto fetch_v = [&](int kb) {
    const bf16_t* vb = Vc + (size_t)(min(kb, max_slot & ~31) >> 5) * (32 * DH) + lane * 8;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) V[ct] = *reinterpret_cast<const u32x4*>(vb + ct * 512);
  };
  fetch_k(w * 32);
  fetch_v(w * 32);
  {
    const float scale = a.scale * 1.4426950408889634f, sg = c4 >= DH / 2 ? 1.f : -1.f;
#pragma unroll
    for (int i = 0; i < QI; ++i) {
      const int col = (i * NW + w) * RPI + lane / LPR;
      float4 x = qx[i];
      if (ROPE) {
        const float4 xp = qp[i], c = qc[i][0], d = qc[i][1];
        x.x = x.x * c.x + sg * (xp.x * c.y); x.y = x.y * c.z + sg * (xp.y * c.w);
        x.z = x.z * d.x + sg * (xp.z * d.y); x.w = x.w * d.z + sg * (xp.w * d.w);
      }
      uint2 qh, ql;
      split2(x.x * scale, x.y * scale, qh.x, ql.x);
      split2(x.z * scale, x.w * scale, qh.y, ql.y);
      if (col < 16) {
        const int to = ((c4 & 31) >> 3) * 16 + col;
        *reinterpret_cast<uint2*>((char*)&lds_q[c4 >> 5][0][to] + (c4 & 4) * 2) = qh;
        *reinterpret_cast<uint2*>((char*)&lds_q[c4 >> 5][1][to] + (c4 & 4) * 2) = ql;
      }
    }
  }
  lds_barrier();
  const int slot = l16 < n_col ? slot0 + (l16 >> lg) : -1;           // this lane's query; -1: none, every key masked
  f32x4 O[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) O[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
  float m_run = NEG, l_run = 0.f;
  for (int kb = w * 32; kb <= max_slot; kb += 32 * NW) {
    f32x4 sc[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int hl = 0; hl < 2; ++hl) {
        const uint4 q = __builtin_bit_cast(uint4, lds_q[t][hl][lane]);
        sc[0] = mfma_bf16(__builtin_bit_cast(uint4, K[0][t]), q, sc[0]);
        sc[1] = mfma_bf16(__builtin_bit_cast(uint4, K[1][t]), q, sc[1]);
      }
    __builtin_amdgcn_sched_barrier(0);
    fetch_k(kb + 32 * NW);
    __builtin_amdgcn_sched_barrier(0);
    const int left = slot - kb - lq * 8;                         // keys 0 .. left of this lane's 8 are valid
    float x[8], p[8], mx = NEG;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      x[e] = e <= left ? sc[e >> 2][e & 3] : NEG;
      mx = fmaxf(mx, x[e]);
    }
    const float mn = fmaxf(m_run, quarter_max(mx)), corr = __builtin_amdgcn_exp2f(m_run - mn);
    m_run = mn;
    l_run *= corr;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) O[ct] *= corr;
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = e <= left ? __builtin_amdgcn_exp2f(x[e] - mn) : 0.f;
    l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    uint4 ph, pl;
    split2(p[0], p[1], ph.x, pl.x);
    split2(p[2], p[3], ph.y, pl.y);
    split2(p[4], p[5], ph.z, pl.z);
    split2(p[6], p[7], ph.w, pl.w);
    if (kb + 31 > max_slot) {                                    // (scalar) zero the values of keys beyond the group's last one
      unsigned keep[4];
      vt_first(max_slot + 1 - kb - lq * 8, keep);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) V[ct][e] &= keep[e];
    }
    unsigned odd = 0;                                            // an infinity or NaN among the values of a block with the group's own keys:
    if (n > 1 && kb + 31 > slot0) {                              // (scalar) an exponent of all ones carries into the sign's place
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) odd |= (V[ct][e] & 0x7f807f80u) + 0x00800080u;
    }
    if (__any((odd & 0x80008000u) != 0)) {                       // (uniform) queries from the first such key on get NaN, the others zeros in its place
      int first = max_slot + 1;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        bool bad = false;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) bad |= ((V[ct][e >> 1] >> (16 * (e & 1))) & 0x7f80u) == 0x7f80u;
        const u64 lanes = __ballot(bad);
        if (lanes) first = min(first, kb + (__builtin_ctzll(lanes) >> 4) * 8 + e);
        __builtin_amdgcn_sched_barrier(0);                       // (registers)
      }
      if (slot >= first) l_run = NAN;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        asm volatile("" : "+v"(V[ct]));                          // (else the test's sums are kept in registers for the next lines)
#pragma unroll
        for (int e = 0; e < 4; ++e) V[ct][e] &= ~(((((V[ct][e] & 0x7f807f80u) + 0x00800080u) & 0x80008000u) >> 15) * 0xffffu);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) O[ct] = mfma_bf16(__builtin_bit_cast(uint4, V[ct]), ph, O[ct]);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) O[ct] = mfma_bf16(__builtin_bit_cast(uint4, V[ct]), pl, O[ct]);
    __builtin_amdgcn_sched_barrier(0);
    fetch_v(kb + 32 * NW);
    __builtin_amdgcn_sched_barrier(0);
  }
  l_run = quarter_sum(l_run);
  if (lq == 0) { s_ml[w][l16][0] = m_run; s_ml[w][l16][1] = l_run; }
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) *reinterpret_cast<f32x4*>(&s_o[w][l16][ct * 16 + lq * 4]) = O[ct];
  lds_barrier();
  bf16_t* __restrict__ ao = (bf16_t*)a.ao;
  for (int idx = tid; idx < n_col * (DH / 4); idx += NW * 64) {
    const int col = idx / (DH / 4), i = idx % (DH / 4) * 4;
    float mn = NEG, den = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) mn = fmaxf(mn, s_ml[q][col][0]);
    f32x4 num = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const float c = __builtin_amdgcn_exp2f(s_ml[q][col][0] - mn);
      den += c * s_ml[q][col][1];
      num += c * *reinterpret_cast<const f32x4*>(&s_o[q][col][i]);
    }
    num *= 1.0f / den;
    *reinterpret_cast<uint2*>(ao + act_idx<bf16_t>(r + col / G, (kvh * G + col % G) * DH + i, a.ao_K)) =
        make_uint2(pk_f16(num[0], num[1]), pk_f16(num[2], num[3]));
  }
}

// A compute unit pulls at most 48 KB/us, so one workgroup needs 21 us for 2000 keys of 128 columns: few rows with long contexts
// share the keys over as many workgroups as the compute units allow, at the price of a merge launch.  Both launches together, one
// workgroup / split, 8 KV heads of 128 columns: 4 rows (split 8) at 1024 keys 19.0 / 13.2 us, 2016 29.9 / 14.6; 16 rows (2) at 1024
// 22.9 / 21.7, 2016 36.7 / 32.5; of 64 columns: 4 rows at 1536 13.7 / 9.7, 2016 16.5 / 10.3; 16 rows at 1536 16.5 / 16.4, 2016 19.7 /
// 18.9.  The line is where a split in two breaks even (16 rows, 128 columns: 768 keys 19.3 / 20.4; a launch works in steps of 256
// keys a workgroup, and from 769 on it is four against two); a split in 8 is ahead from about 256 KB on.
int attn_split(int dh, int kvh, int rows, int ctx_bound) {
  if ((long long)kvh * rows > SPLIT_WGS / 2 || ctx_bound < 512 || (size_t)ctx_bound * dh * 4 < 400 * 1024) return 1;
  return std::min(8, SPLIT_WGS / (kvh * rows));
}

// Prefill of grouped queries: whether four waves share the keys and values of a KV head.  Below one wave per SIMD in the whole launch (1024 pairs
// of heads x 16 entries) each has the memory to itself, and the workgroup's start and the waves without entries of a run cost what
// nothing gives back; likewise where the longest prompt is short, five times as far at 64 columns (half the bytes of a key, and half the work to
// hide the start behind), and where the prompts cover less than half of a workgroup's 128 / G entries in the mean: it goes through its
// runs one after the other.  us, one wave / shared, heads and KV heads, columns:
//   shared: four of 512, 32 over 8, 128: 48 / 43; four of 1000, 16 over 8, 128: 73 / 65; eight of 512, 32 over 8, 128: 73 / 66; three of 1500, 32 over 4, 64: 90 / 76
//   not: one of 300, 16 over 2, 128: 16.8 / 18.3; one of 600, 28.2 / 28.5; six of 768, 32 over 8, 64: 57 / 62; 20 of 200, 16 over 8, 128: 28 / 30;
//        one of 1030 and 100 of 10, 12 over 6, 64: 32 / 41, 16 over 8, 128: 51 / 58
// Of 948 such points (1 - 300 prompts of 9 - 2000 entries, 12 shapes) the rule shares 299, 12 % faster in the mean; two of them are slower for
// it, by 2 and 4 %.
bool attn_shared(int dh, int H, int KVH, int entries, int ctx_bound, int run_len) {
  const int G = H / KVH;
  return G > 1 && (long long)(H / 2) * ((entries + 15) / 16) >= 1024 && (long long)ctx_bound * G >= (dh == 64 ? 7168 : 1536) && (long long)run_len * G >= 64;
}

template <int DH>
static void launch_attn_bf16(const AttnArgs& a, int G, int max_rows, int ctx_bound, int run_len, hipStream_t s) {
  if (a.phase == 1) {          // append only
    hipLaunchKernelGGL((k_kv_append_bf16<DH>), dim3(a.KVH, (max_rows + 7) / 8), dim3(64), 0, s, a);
    return;
  }
  if (a.phase == 3) {          // attend-only over runs of consecutive positions of one row: the matrix-core kernel
    if (attn_shared(DH, a.H, a.KVH, max_rows, ctx_bound, run_len))
      hipLaunchKernelGGL((k_attn_mfma_shared_bf16<DH>), dim3(a.KVH, (max_rows + 128 / G - 1) / (128 / G)), dim3(256), 0, s, a);
    else if (G > 1) hipLaunchKernelGGL((k_attn_mfma_bf16<DH, true>), dim3(a.H / 2, (max_rows + 15) / 16), dim3(64), 0, s, a);
    else hipLaunchKernelGGL((k_attn_mfma_bf16<DH, false>), dim3(a.H, (max_rows + 31) / 32), dim3(64), 0, s, a);
    return;
  }
  // NW = waves per workgroup that share one (row, KV head)'s keys: 8 when the launch has no more workgroups than
  // the chip has compute units and the contexts are long, else 4
  dim3 grid(a.KVH, max_rows);
  const bool wide = (long long)a.KVH * max_rows <= 256 && ctx_bound >= 512;
  if (a.phase == 2) {          // attend-only, short runs
#define SPRINTER_RUNS(NW, ROPE) hipLaunchKernelGGL((k_attn_runs_bf16<DH, NW, ROPE>), grid, dim3(NW * 64), 0, s, ATTN_VALUES(a, max_rows, 2))
    if (a.use_rope) { if (wide) SPRINTER_RUNS(8, true); else SPRINTER_RUNS(4, true); }
    else { if (wide) SPRINTER_RUNS(8, false); else SPRINTER_RUNS(4, false); }
#undef SPRINTER_RUNS
    return;
  }
  // 64 columns and 129 - 256 keys: eight waves take one step where four take two, and one workgroup per compute unit leaves their loads alone.  us per launch, 4 / 8
  // waves: 25 heads, 130 keys, 1 row 5.14 / 4.68, 190 keys, 5 rows 5.35 / 4.88, 12 heads, 150 keys, 16 rows 6.40 / 6.22, 8 KV heads, 230 keys, 1 row 5.12 / 4.66; but two
  // steps for three, 300 keys, 8 KV heads, 4 rows 5.95 / 6.58, 16 rows 6.09 / 6.86, and at 128 columns 280 keys, 32 heads, 3 rows 7.90 / 8.84.
  const bool one_step = DH == 64 && (long long)a.KVH * max_rows <= 256 && ctx_bound > 128 && ctx_bound <= 256;
  const int split = attn_split(DH, a.KVH, max_rows, ctx_bound);
  grid.z = split;
#define SPRINTER_DEC(NW, NV, ROPE) hipLaunchKernelGGL((k_attn_dec_bf16<DH, NW, NV, ROPE>), grid, dim3(NW * 64), 0, s, ATTN_VALUES(a, split, 2), a.split)
#define SPRINTER_DEC_NW(NV, ROPE) do { if (wide || one_step || split > 1) SPRINTER_DEC(8, NV, ROPE); else SPRINTER_DEC(4, NV, ROPE); } while (0)
  if (G <= 4) { if (a.use_rope) SPRINTER_DEC_NW(1, true); else SPRINTER_DEC_NW(1, false); }
  else { if (a.use_rope) SPRINTER_DEC_NW(2, true); else SPRINTER_DEC_NW(2, false); }
#undef SPRINTER_DEC_NW
#undef SPRINTER_DEC
  if (split > 1) hipLaunchKernelGGL((k_attn_merge<DH>), dim3(a.H, max_rows), dim3(DH), 0, s, a, split);
}

template <int DH>
static void launch_attn_f32(const AttnArgs& a, int max_rows, hipStream_t s) {
  const dim3 grid(a.KVH, max_rows);
#define SPRINTER_AF32(G) do { if (a.use_rope) hipLaunchKernelGGL((k_attn_f32<DH, G, true>), grid, dim3(256), 0, s, ATTN_VALUES(a, a.phase, 4)); \
                              else hipLaunchKernelGGL((k_attn_f32<DH, G, false>), grid, dim3(256), 0, s, ATTN_VALUES(a, a.phase, 4)); } while (0)
  switch (a.G) {
    case 1: SPRINTER_AF32(1); break;
    case 2: SPRINTER_AF32(2); break;
    case 4: SPRINTER_AF32(4); break;
    default: SPRINTER_AF32(8); break;
  }
#undef SPRINTER_AF32
}

void launch_attention(int dtype, const ModelDims& md, const float* y, const float* rope, const RowDesc& rd,
                      void* kcache, void* vcache, size_t layer_off, int ctx_bound, int max_seq, void* ao,
                      int max_rows, float* split, hipStream_t s, int phase, int run_len) {
  AttnArgs a;
  a.phase = (phase == 3 && dtype == 0) ? 2 : phase;      // the run-sharing kernel exists for bf16 only
  a.y = y; a.rope = rope; a.rd = rd; a.kcache = kcache; a.vcache = vcache; a.layer_off = layer_off;
  a.H = md.H; a.KVH = md.KVH; a.G = md.H / md.KVH; a.lg = __builtin_ctz(a.G); a.dqkv = md.dqkv; a.max_seq = max_seq; a.use_rope = md.arch == 1;
  a.scale = 1.0f / sqrtf((float)md.dh);
  a.ao = ao; a.ao_K = md.H * md.dh; a.split = split;
  int G = md.H / md.KVH;
  if (dtype == 0) {
    if (md.dh == 64) launch_attn_f32<64>(a, max_rows, s); else launch_attn_f32<128>(a, max_rows, s);
  } else {
    if (md.dh == 64) launch_attn_bf16<64>(a, G, max_rows, ctx_bound, run_len, s); else launch_attn_bf16<128>(a, G, max_rows, ctx_bound, run_len, s);
  }
}

}  // namespace sprinter
