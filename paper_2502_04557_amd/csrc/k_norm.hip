// HIP kernels of the batched SPRINTER decode step for gfx950 (wave64, MFMA): weight packing, embedding
// and the layer norms.  One decode step (Alg. 2 of the paper, run for B rows in lock step):
//   draft forward -> LM head + Gumbel-max sample -> verifier + threshold ->
//   compaction of rejected rows -> target forward on those rows -> sample -> scatter back.
// Every kernel reads the number of active rows from device memory; the launch shapes are upper
// bounds the host chooses.
#include "dev.h"
#include <algorithm>
#include <cstring>
#include <type_traits>

namespace sprinter {

// ================================================================ packing
// [N, K] row-major bf16 -> operand tiles of float16 (zero padded to 16 rows x 32 k).  A bf16 value has 8 significant
// bits and converts exactly above 2^-14; smaller ones round to the float16 subnormal grid (2^-24 apart).
__global__ __launch_bounds__(256) void k_pack_bf16(const bf16_t* __restrict__ w, uint4* __restrict__ out, int N, int K,
                                                   int Kt, size_t total) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  int lane = (int)(i & 63);
  size_t tile = i >> 6;
  int kt = (int)(tile % Kt);
  int nt = (int)(tile / Kt);
  int n = nt * 16 + (lane & 15);
  int k0 = kt * 32 + (lane >> 4) * 8;
  uint4 v = make_uint4(0, 0, 0, 0);
  if (n < N) {
    if (k0 + 8 <= K) {
      v = *reinterpret_cast<const uint4*>(w + (size_t)n * K + k0);   // K % 8 == 0 keeps this aligned
    } else if (k0 < K) {
      bf16_t t[8];
      for (int e = 0; e < 8; ++e) t[e] = (k0 + e < K) ? w[(size_t)n * K + k0 + e] : (bf16_t)0;
      v = *reinterpret_cast<uint4*>(t);
    }
  }
  const unsigned wd[4] = {v.x, v.y, v.z, v.w};
  unsigned o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = pk_f16(__uint_as_float(wd[e] << 16), __uint_as_float(wd[e] & 0xffff0000u));
  out[i] = make_uint4(o[0], o[1], o[2], o[3]);
}
void launch_pack_bf16(const void* w, void* out, int N, int K, hipStream_t s) {
  int Kt = (K + 31) / 32, Nt = (N + 15) / 16;
  size_t total = (size_t)Nt * Kt * 64;
  hipLaunchKernelGGL(k_pack_bf16, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const bf16_t*)w,
                     (uint4*)out, N, K, Kt, total);
}

__global__ __launch_bounds__(256) void k_fill_zero(uint4* p, size_t n16) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  size_t stride = (size_t)gridDim.x * 256;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}
void launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  size_t n16 = bytes / 16;
  if (!n16) return;
  unsigned grid = (unsigned)((n16 + 255) / 256);
  if (grid > 4096) grid = 4096;
  hipLaunchKernelGGL(k_fill_zero, dim3(grid), dim3(256), 0, s, (uint4*)p, n16);
}

// =================================================================== norm
// LayerNorm (arch 0) / RMSNorm (arch 1), two-pass statistics: one row per workgroup, one thread per 8 consecutive columns
// (bf16 mode: one 16-byte slot of a float16 operand tile), so the row, gain and offset are requested with six 16-byte
// loads per thread before anything is waited for and the result leaves as one or two 16-byte stores.  d <= 8192.
// NI = 2048-column blocks per row (1, 2 or 4); SH = 0, or the most partial products a pending update of the
// residual stream may consist of (1, 2, 4 or 8; one share, which float32 mode leaves and bf16 mode at up to 16 rows of more than 4096 columns, with the loads of four:
// 4096 columns, 8 rows 3.25 -> 3.70 us; two, which most O-projections of 9 - 16 rows leave: 1600 columns, 6 rows 3.0 -> 3.3, 4096 rows of 768 11.1 -> 12.6): the row is then h + bias + share 0 + share 1 + ..., added in that
// order, written back and normalised.  The partial loads are issued with the others, before the row count
// is known, with clamped share indices and the surplus selected away - no branch, no second memory round.
// SH = -1: the first norm of a forward; the row is the token's embedding (+ the position's) and starts the residual stream
// (an embedding launch of its own cost 1.9 - 4.8 us).  The rotary factors of all rows come from workgroups of their own behind the
// rows' (n_rows_grid of them): their double-precision pow / cos / sin take 2.5 us, next to the rows' norm instead of ahead of it.
// The row of workgroup id.  An operand tile holds 16 bytes of each of 16 rows side by side, and workgroups go round-robin over the 8
// XCDs: in order, every 128-byte line was written in pieces by 8 L2s.  Of 128 workgroups, the 16 of an XCD take the 16 rows of a tile.
// us at 4096 / 1785 / 512 rows, in order -> so: 4096 columns 39.7 / 20.3 / 6.3 -> 28.6 / 12.5 / 4.7, 1600 with 4 shares 34.1 / 15.4 / 5.7 ->
// 28.1 / 13.7 / 4.7; 199 rows of 4096 4.0 -> 3.2.
__device__ __forceinline__ int norm_row(int id, int rows) {
  return id < (rows & ~127) ? (id & ~127) + (id & 7) * 16 + ((id >> 3) & 15) : id;
}
template <typename AT, int ARCH, int NI, int SH>
__global__ __launch_bounds__(256) void k_norm(const float* __restrict__ h, const float* __restrict__ g, const float* __restrict__ b,
                                                   const float* __restrict__ part, const float* __restrict__ part_bias, int d, int n_rows_grid, int shares, float eps,
                                                   const int* __restrict__ n_rows, AT* __restrict__ act_out, float* __restrict__ f32_out, size_t part_stride,
                                                   std::conditional_t<(SH < 0), EmbedSource, Nothing> emb) {
  const NormPending pend{part, part_stride, shares, part_bias};
  __shared__ float s_sum[4], s_sq[4];
  const int r = norm_row(blockIdx.x, n_rows_grid), tid = threadIdx.x;
  if constexpr (SH < 0 && ARCH == 1) {
    if (__builtin_expect(r >= n_rows_grid, 0)) {
      const int i = (r - n_rows_grid) * 256 + tid, half = emb.dh >> 1;
      if (i / half < *n_rows) rope_factors(emb, i / half, i % half);
      return;
    }
  }
  const float4* __restrict__ x4 = reinterpret_cast<const float4*>(h + (size_t)r * d);
  const float4* __restrict__ g4 = reinterpret_cast<const float4*>(g);
  const float4* __restrict__ b4 = reinterpret_cast<const float4*>(b);
  const int n_chunks = d >> 3;                       // d is a multiple of 8
  float x[NI][8], gg[NI][8], bb[NI][8];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = min(tid + i * 256, n_chunks - 1);  // clamped: no branch around the loads
    if (SH >= 0) { *reinterpret_cast<float4*>(&x[i][0]) = x4[2 * c]; *reinterpret_cast<float4*>(&x[i][4]) = x4[2 * c + 1]; }
    *reinterpret_cast<float4*>(&gg[i][0]) = g4[2 * c]; *reinterpret_cast<float4*>(&gg[i][4]) = g4[2 * c + 1];
    if (ARCH == 0) { *reinterpret_cast<float4*>(&bb[i][0]) = b4[2 * c]; *reinterpret_cast<float4*>(&bb[i][4]) = b4[2 * c + 1]; }
  }
  if constexpr (SH < 0) {
    const int tok = min(max(emb.rd.tok[r], 0), emb.V - 1);   // (an out-of-vocabulary id must not become a wild read)
    const int pos = max(emb.rd.pos[r], 0);
    const AT* __restrict__ e = (const AT*)emb.tok_emb + (size_t)tok * d;
    const AT* __restrict__ p = emb.pos_emb ? (const AT*)emb.pos_emb + (size_t)min(pos, emb.max_pos - 1) * d : nullptr;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = min(tid + i * 256, n_chunks - 1);
      load_row(e + c * 8, x[i]);
      if (p) {
        float pv[8];
        load_row(p + c * 8, pv);
#pragma unroll
        for (int k = 0; k < 8; ++k) x[i][k] += pv[k];
      }
    }
  }
  if constexpr (SH > 0) {
    const float4* __restrict__ pb4 = reinterpret_cast<const float4*>(pend.bias ? pend.bias : g);
    const bool has_bias = pend.bias != nullptr;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = min(tid + i * 256, n_chunks - 1);
      float4 p0[SH + 1], p1[SH + 1];
      p0[0] = pb4[2 * c]; p1[0] = pb4[2 * c + 1];
#pragma unroll
      for (int q = 0; q < SH; ++q) {
        const float4* p4 = reinterpret_cast<const float4*>(pend.part + (size_t)min(q, pend.shares - 1) * pend.stride + (size_t)r * d);
        p0[q + 1] = p4[2 * c]; p1[q + 1] = p4[2 * c + 1];
      }
#pragma unroll
      for (int q = 0; q <= SH; ++q) {                // fixed order: bias, share 0, share 1, ...
        const bool on = q == 0 ? has_bias : q - 1 < pend.shares;
        x[i][0] += on ? p0[q].x : 0.f; x[i][1] += on ? p0[q].y : 0.f; x[i][2] += on ? p0[q].z : 0.f; x[i][3] += on ? p0[q].w : 0.f;
        x[i][4] += on ? p1[q].x : 0.f; x[i][5] += on ? p1[q].y : 0.f; x[i][6] += on ? p1[q].z : 0.f; x[i][7] += on ? p1[q].w : 0.f;
      }
    }
  }
  if (r >= *n_rows) return;
  if (SH != 0) {
    float* hrow = const_cast<float*>(h) + (size_t)r * d;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = tid + i * 256;
      if (c < n_chunks) {
        *reinterpret_cast<float4*>(hrow + c * 8) = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
        *reinterpret_cast<float4*>(hrow + c * 8 + 4) = make_float4(x[i][4], x[i][5], x[i][6], x[i][7]);
      }
    }
  }
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const bool ok = tid + i * 256 < n_chunks;
#pragma unroll
    for (int e = 0; e < 8; ++e) { x[i][e] = ok ? x[i][e] : 0.f; sum += x[i][e]; }
  }
  float mean = 0.f;
  if (ARCH == 0) mean = block_total256(sum, s_sum) / (float)d;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const bool ok = tid + i * 256 < n_chunks;
#pragma unroll
    for (int e = 0; e < 8; ++e) { const float c = ok ? x[i][e] - mean : 0.f; sq += c * c; }
  }
  const float var = block_total256(sq, s_sq) / (float)d;
  const float rstd = 1.0f / sqrtf(var + eps);
  const int Kt = (d + 31) >> 5;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = tid + i * 256;
    if (c < n_chunks) {
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        o[e] = (x[i][e] - mean) * rstd * gg[i][e];
        if (ARCH == 0) o[e] += bb[i][e];
      }
      const int k = c * 8;
      if constexpr (sizeof(AT) == 2) {
        const uint4 ov = make_uint4(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]), pk_f16(o[4], o[5]), pk_f16(o[6], o[7]));
        const size_t slot = ((size_t)(r >> 4) * Kt + (k >> 5)) * 512 + ((((k & 31) >> 3) << 4) + (r & 15)) * 8;
        *reinterpret_cast<uint4*>(act_out + slot) = ov;
      } else {
        *reinterpret_cast<float4*>(act_out + (size_t)r * d + k) = make_float4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<float4*>(act_out + (size_t)r * d + k + 4) = make_float4(o[4], o[5], o[6], o[7]);
      }
      if (f32_out) {
        *reinterpret_cast<float4*>(f32_out + (size_t)r * d + k) = make_float4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<float4*>(f32_out + (size_t)r * d + k + 4) = make_float4(o[4], o[5], o[6], o[7]);
      }
    }
  }
}

// The same for the many rows of a prefill pass (bf16 mode, activations only, nothing pending), a row per wave and four rows per workgroup: no barrier
// stands between a row's loads and its statistics, and the float16 rows leave through LDS, four rows of a tile side by side - 64
// bytes to an address, where a row alone has 16.  The columns, and with them the order of every sum, are those of k_norm: chunk
// 256 i + 64 v + lane is thread 64 v + lane's i-th there.  LDS slot of (chunk c, row r): 4 c + (r ^ (c / 4 % 4)), which spreads a wave's
// stores over the banks.  What bounds it: 100 MB at 4096 x 4096 take 17 us at the rate of a copy, it 24.
template <int ARCH, int NI>
__global__ __launch_bounds__(256) void k_norm_rows(const float* __restrict__ h, const float* __restrict__ g, const float* __restrict__ b,
                                                   float eps, int d, const int* __restrict__ n_rows, bf16_t* __restrict__ act_out, int groups) {
  extern __shared__ __align__(16) uint4 tile[];
  const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), id = blockIdx.x;
  // the 4 workgroups of a row tile on one XCD
  const int grp = id < (groups & ~31) ? (id & ~31) + (id & 7) * 4 + ((id >> 3) & 3) : id, r0 = grp * 4, r = r0 + w;
  const int n = *n_rows, n_chunks = d >> 3;
  if (r0 >= n) return;
  if (r < n) {                                       // (scalar)
    const float* __restrict__ hrow = h + (size_t)r * d;
    float x[NI][4][8];
    auto chunk = [&](int i, int v) { return min(i * 256 + v * 64 + lane, n_chunks - 1); };
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) load_row(hrow + chunk(i, v) * 8, x[i][v]);
    auto total = [&](const float (&s)[4]) {
      float t[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) t[v] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wave_total(s[v])), 63));
      return ((t[0] + t[1]) + t[2]) + t[3];
    };
    float s[4] = {0.f, 0.f, 0.f, 0.f}, mean = 0.f;
    if (ARCH == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) s[v] += i * 256 + v * 64 + lane < n_chunks ? x[i][v][e] : 0.f;
      mean = total(s) / (float)d;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      s[v] = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) { const float c = i * 256 + v * 64 + lane < n_chunks ? x[i][v][e] - mean : 0.f; s[v] += c * c; }
    }
    const float rstd = 1.0f / sqrtf(total(s) / (float)d + eps);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = i * 256 + v * 64 + lane;
        float gg[8], bb[8], o[8];
        load_row(g + chunk(i, v) * 8, gg);
        if (ARCH == 0) load_row(b + chunk(i, v) * 8, bb);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          o[e] = (x[i][v][e] - mean) * rstd * gg[e];
          if (ARCH == 0) o[e] += bb[e];
        }
        if (c < n_chunks) tile[c * 4 + (w ^ ((c >> 2) & 3))] = make_uint4(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]), pk_f16(o[4], o[5]), pk_f16(o[6], o[7]));
      }
  }
  __syncthreads();
  const int Kt = (d + 31) >> 5, row = tid & 3;
  if (r0 + row >= n) return;
  for (int c = tid >> 2; c < n_chunks; c += 64) {
    const size_t slot = ((size_t)(r0 >> 4) * Kt + (c >> 2)) * 512 + (((c & 3) << 4) + (r0 & 15) + row) * 8;
    *reinterpret_cast<uint4*>(act_out + slot) = tile[c * 4 + (row ^ ((c >> 2) & 3))];
  }
}

// k_norm_rows / k_norm, us: 4096 rows of 4096 columns 24.2 / 28.7, 2048 12.1 / 15.3, 768 5.8 / 6.2; 1785 rows of 4096 10.4 / 12.5, 2048 6.1 / 6.5, but 1600
// 6.1 / 5.8; 1000 rows of 4096 7.6 / 7.2: too few waves for their loads.  (With shares to add it is 5 - 20 % slower at any size: k_norm
// requests them all together.)
static bool norm_takes_rows(int d, int rows) { return rows >= 3072 || (rows >= 1536 && d >= 2048); }
template <typename AT, int ARCH, int NI>
static void launch_norm_ni(const float* h, const float* g, const float* b, float eps, int d, const int* n_rows,
                           void* act_out, float* f32_out, int max_rows, hipStream_t s, const NormPending& np, const EmbedSource* emb) {
  EmbedSource es;
  memset(&es, 0, sizeof es);
  if (emb) es = *emb;
  if constexpr (sizeof(AT) == 2) {
    if (!emb && !f32_out && np.shares <= 0 && norm_takes_rows(d, max_rows)) {
      const int groups = (max_rows + 3) / 4;
      hipLaunchKernelGGL((k_norm_rows<ARCH, NI>), dim3(groups), dim3(256), (size_t)d * 8, s, h, g, b, eps, d, n_rows, (bf16_t*)act_out, groups);
      return;
    }
  }
  const int rope_wgs = es.rope ? (int)(((size_t)max_rows * (es.dh / 2) + 255) / 256) : 0;
#define SPRINTER_NORM(SH) hipLaunchKernelGGL((k_norm<AT, ARCH, NI, SH>), dim3(max_rows), dim3(256), 0, s, h, g, b, np.part, np.bias, d, max_rows, np.shares, eps, n_rows, (AT*)act_out, f32_out, np.stride, Nothing{})
  if (emb) hipLaunchKernelGGL((k_norm<AT, ARCH, NI, -1>), dim3(max_rows + rope_wgs), dim3(256), 0, s, h, g, b, nullptr, nullptr, d, max_rows, 0, eps, n_rows, (AT*)act_out, f32_out, 0, es);
  else if (np.shares <= 0) SPRINTER_NORM(0);
  else if (np.shares == 1) SPRINTER_NORM(1);
  else if (np.shares == 2) SPRINTER_NORM(2);
  else if (np.shares <= 4) SPRINTER_NORM(4);
  else SPRINTER_NORM(8);
#undef SPRINTER_NORM
}
template <typename AT, int ARCH>
static void launch_norm_arch(const float* h, const float* g, const float* b, float eps, int d, const int* n_rows,
                             void* act_out, float* f32_out, int max_rows, hipStream_t s, const NormPending& np, const EmbedSource* emb) {
  if (d <= 2048) launch_norm_ni<AT, ARCH, 1>(h, g, b, eps, d, n_rows, act_out, f32_out, max_rows, s, np, emb);
  else if (d <= 4096) launch_norm_ni<AT, ARCH, 2>(h, g, b, eps, d, n_rows, act_out, f32_out, max_rows, s, np, emb);
  else launch_norm_ni<AT, ARCH, 4>(h, g, b, eps, d, n_rows, act_out, f32_out, max_rows, s, np, emb);
}

void launch_norm(int dtype, int arch, const float* h, const float* g, const float* b, float eps, int d,
                 const int* n_rows, void* act_out, float* f32_out, int max_rows, hipStream_t s,
                 const NormPending* pend, const EmbedSource* emb) {
  NormPending np;
  memset(&np, 0, sizeof np);
  if (pend) np = *pend;
#define NORM_CASE(AT, ARCH) launch_norm_arch<AT, ARCH>(h, g, b, eps, d, n_rows, act_out, f32_out, max_rows, s, np, emb)
  if (dtype == 0) { if (arch == 0) NORM_CASE(float, 0); else NORM_CASE(float, 1); }
  else            { if (arch == 0) NORM_CASE(bf16_t, 0); else NORM_CASE(bf16_t, 1); }
#undef NORM_CASE
}

}  // namespace sprinter
