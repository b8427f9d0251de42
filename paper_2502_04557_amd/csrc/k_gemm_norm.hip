// HIP kernel of the batched SPRINTER decode step for gfx950: QKV projection and FFN-up for a few rows, with the layer norm
// (and the residual update or embedding before it) folded into the same launch.
#include "gemm.h"
#include <algorithm>
#include <cstring>

namespace sprinter {

// At a handful of rows a step is a chain of short dependent launches, and the norm is two of a layer's seven: 3 - 4 us each
// for a few KiB of work.  Here every workgroup of the product that follows normalises the rows for itself: it requests the
// weight tiles of its first k tiles, then reads the residual rows and the pending partial products (or the embeddings), adds
// them in the order of k_norm, takes the statistics in two passes, and leaves the normalised rows in LDS, from where the
// matrix instructions take them.  Workgroup 0 also writes the updated residual rows - to the other of two buffers, since its
// neighbours are still reading this one.  What it costs is R d (1 + shares) floats per workgroup through L2 next to its own
// weights, so it is taken only while that stays small (gemm_takes_norm).  In a chain - partial product, norm, product - as three
// launches against two, at 1 / 2 / 3 / 4 rows, us: d = 1600, FFN-down in 4 shares, QKV 4800: 14.9 -> 13.1 / 13.4 / 14.2 / 15.1; O-proj
// in 2, FFN-up 6400: 12.7 -> 10.7 / 11.4 / 12.0 / 12.7; d = 2048 (RMS), 4 shares, QKV 3072: 16.1 -> 13.5 / 14.2 / 14.9 / 15.5; 2 shares,
// 2 x 8192: 20.7 -> 18.5 / 19.1 / 19.3 / 19.8; d = 768, 4 shares, QKV 2304: 12.0 -> 7.7 / 8.3 / 9.1 / 9.7; d = 512, 3 shares, 1024:
// 11.6 -> 8.0 / 7.5 / 7.6 / 8.1.  Fewer shares cost the partial product more than they save here (1600, 4 rows: 15.1 with 4, 16.2 with 2).
// Up to R rows.  Four and less: thread t takes float4 t of every row (d <= 2048), so gain, offset and bias are fetched once.  More (d <= 512): four
// groups of 128 threads take R / 4 rows each, float4 t % 128 of them.
template <typename AT, int R, int NTW, int EPI>
__global__ __launch_bounds__(512) void k_gemm_norm(GemmArgs a, NormFusion f) {
  constexpr bool BF = sizeof(AT) == 2;                  // bf16 mode: float16 operand tiles; else float32 rows
  constexpr bool DUAL = (EPI == EPI_SWIGLU), ACT_OUT = BF && (EPI == EPI_GELU || EPI == EPI_SWIGLU);
  constexpr int NW = NTW * (DUAL ? 2 : 1), NI4 = NW * 4, U = 8;   // weight tiles per k tile; k tiles (16-k groups) in flight
  constexpr int RG = R > 4 ? 4 : 1, RT = (R + RG - 1) / RG, WR = 8 / RG;   // groups of threads, rows per thread, waves per row
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) float s_stat[2][R][WR];
  __shared__ float red[8 * NI4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), l16 = lane & 15, lq = lane >> 4;
  const int nt0 = blockIdx.x * NTW, d = a.K;
  if constexpr (EPI == EPI_F32) {
    if (__builtin_expect(nt0 >= a.n_tiles, 0)) {        // QKV of a first layer with rotary positions: one workgroup more for the rows' factors
      const int half = f.emb.dh >> 1;
      for (int i = tid; i < a.rows_live * half; i += 512) rope_factors(f.emb, i / half, i % half);
      return;
    }
  }
  // ---- this wave's share of K: k tiles w, w + 8, .. (bf16) or 16-k groups [g0, g1) (float32); first weights requested
  const int n_k = BF ? a.Kt : d >> 4;
  const int g0 = BF ? w : n_k * w / 8, g1 = BF ? n_k : n_k * (w + 1) / 8, gs = BF ? 8 : 1;
  const uint4* wp[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) {
    const void* W = DUAL && j >= NTW ? a.W2 : a.W;
    const int nt = min(nt0 + (j % NTW), a.n_tiles - 1);
    wp[j] = BF ? (const uint4*)W + (size_t)nt * a.Kt * 64 + lane
               : (const uint4*)((const float*)W + (size_t)min(nt * 16 + l16, a.N - 1) * d + lq * 4);
  }
  uint4 wv[U][NW];
  auto load_weights = [&](int g) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g + u * gs < g1) {                            // (scalar; the tiles beyond the share are skipped below too)
#pragma unroll
        for (int j = 0; j < NW; ++j) wv[u][j] = wp[j][(size_t)(g + u * gs) * (BF ? 64 : 4)];
      }
  };
  load_weights(g0);
  // this thread's output element: (row m, column c of the workgroup's 16 NTW columns), as in k_gemm16 / k_gemm_f32
  int m, c;
  if (ACT_OUT) { m = (tid >> 3) & 15; c = (tid >> 7) * 8 + (tid & 7); }
  else { m = tid / (16 * NTW); c = tid % (16 * NTW); }
  const int n = nt0 * 16 + c;
  const bool out_ok = tid < NTW * 256 && m < a.rows_live && n < a.N;
  const float pbias = (out_ok && a.bias) ? a.bias[n] : 0.f;
  // ---- residual rows
  const int n4 = d >> 2, col = tid % (512 / RG), q4 = min(col, n4 - 1), r0 = w / WR * RT;   // this thread's rows: r0 .. (scalar)
  const bool mine = col < n4;
  const float4 gg = reinterpret_cast<const float4*>(f.g)[q4];
  float4 bb = make_float4(0.f, 0.f, 0.f, 0.f), pb = bb, x[RT];
  if (f.b) bb = reinterpret_cast<const float4*>(f.b)[q4];
  if (f.emb.tok_emb) {                                  // first norm of a forward: the token's (and the position's) embedding
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int r = min(r0 + i, a.rows_live - 1);
      const int tok = min(max(f.emb.rd.tok[r], 0), f.emb.V - 1), pos = max(f.emb.rd.pos[r], 0);
      const AT* __restrict__ e = (const AT*)f.emb.tok_emb + (size_t)tok * d;
      const AT* __restrict__ p = f.emb.pos_emb ? (const AT*)f.emb.pos_emb + (size_t)min(pos, f.emb.max_pos - 1) * d : nullptr;
      float ev[4], pv[4] = {0.f, 0.f, 0.f, 0.f};
      load_row(e + q4 * 4, ev);
      if (p) load_row(p + q4 * 4, pv);
      x[i] = make_float4(ev[0] + pv[0], ev[1] + pv[1], ev[2] + pv[2], ev[3] + pv[3]);
    }
  } else {
    if (f.pend.bias) pb = reinterpret_cast<const float4*>(f.pend.bias)[q4];
    float4 p[RT][4];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const size_t q = (size_t)min(r0 + i, a.rows_live - 1) * n4 + q4;
      x[i] = reinterpret_cast<const float4*>(f.h_in)[q];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (s < f.pend.shares) p[i][s] = reinterpret_cast<const float4*>(f.pend.part + (size_t)s * f.pend.stride)[q];   // (scalar test)
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) {                       // fixed order: bias, share 0, share 1, ...
      x[i].x += pb.x; x[i].y += pb.y; x[i].z += pb.z; x[i].w += pb.w;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (s < f.pend.shares) { x[i].x += p[i][s].x; x[i].y += p[i][s].y; x[i].z += p[i][s].z; x[i].w += p[i][s].w; }
    }
  }
  if (blockIdx.x == 0 && mine) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
      if (r0 + i < a.rows_live) reinterpret_cast<float4*>(f.h_out)[(size_t)(r0 + i) * n4 + col] = x[i];
  }
  // ---- statistics: the wave (DPP only), then every thread adds the 8 waves' sums.  No shuffles through LDS and one store
  // block for all rows: a wave-wide butterfly per row, each waited for on its own, was 0.3 us a row.
  float part[RT];
  auto row_sums = [&](int slot) {
#pragma unroll
    for (int i = 0; i < RT; ++i) part[i] = wave_total(part[i]);
    if (lane == 63) {
#pragma unroll
      for (int i = 0; i < RT; ++i) if (r0 + i < a.rows_live) s_stat[slot][r0 + i][w % WR] = part[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const float* st = s_stat[slot][min(r0 + i, a.rows_live - 1)];
      if constexpr (RG == 1) {
        const float4 u = *reinterpret_cast<const float4*>(st), v = *reinterpret_cast<const float4*>(st + 4);
        part[i] = (((u.x + u.y) + (u.z + u.w)) + ((v.x + v.y) + (v.z + v.w)));
      } else {
        part[i] = st[0] + st[1];                        // (the same sum: the other waves' are zero where d <= 512)
      }
    }
  };
  if (f.arch == 0) {
#pragma unroll
    for (int i = 0; i < RT; ++i) part[i] = mine ? (x[i].x + x[i].y) + (x[i].z + x[i].w) : 0.f;
    row_sums(0);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const float mean = part[i] / (float)d;
      x[i].x -= mean; x[i].y -= mean; x[i].z -= mean; x[i].w -= mean;
    }
  }
#pragma unroll
  for (int i = 0; i < RT; ++i) part[i] = mine ? (x[i].x * x[i].x + x[i].y * x[i].y) + (x[i].z * x[i].z + x[i].w * x[i].w) : 0.f;
  row_sums(1);
  // ---- normalised rows to LDS: float16 operand slots [k / 8][row] of 16 bytes, or float32 rows (4 floats of padding)
  if (mine) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const float rstd = 1.0f / sqrtf(part[i] / (float)d + f.eps);
      const float o0 = x[i].x * rstd * gg.x + bb.x, o1 = x[i].y * rstd * gg.y + bb.y;
      const float o2 = x[i].z * rstd * gg.z + bb.z, o3 = x[i].w * rstd * gg.w + bb.w;
      const int r = r0 + i;
      if (r >= a.rows_live) continue;                   // (scalar)
      if (BF) *reinterpret_cast<uint2*>(smem + ((size_t)(col >> 1) * R + r) * 16 + (col & 1) * 8) = make_uint2(pk_f16(o0, o1), pk_f16(o2, o3));
      else *reinterpret_cast<float4*>(smem + ((size_t)r * (d + 4) + col * 4) * 4) = make_float4(o0, o1, o2, o3);
    }
  }
  __syncthreads();
  // ---- product
  const int xrow = min(l16, a.rows_live - 1);        // (lanes of absent rows repeat the last one; their outputs are dropped)
  f32x4 acc[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int g = g0; g < g1; g += U * gs) {
    if (g != g0) load_weights(g);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (g + u * gs < g1) {                            // (scalar)
        if constexpr (BF) {
          const uint4 xv = *reinterpret_cast<const uint4*>(smem + ((size_t)((g + u * 8) * 4 + lq) * R + xrow) * 16);
#pragma unroll
          for (int j = 0; j < NW; ++j) acc[j] = mfma_f16(xv, wv[u][j], acc[j]);
        } else {
          const float4 xv = *reinterpret_cast<const float4*>(smem + ((size_t)xrow * (d + 4) + (g + u) * 16 + lq * 4) * 4);
#pragma unroll
          for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32((&xv.x)[e], __uint_as_float((&wv[u][j].x)[e]), acc[j], 0, 0, 0);
        }
      }
  }
#pragma unroll
  for (int j = 0; j < NW; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((size_t)w * NI4 + j * 4 + v) * 64 + lane] = acc[j][v];
  __syncthreads();
  if (!out_ok) return;
  const int it = (c >> 4) * 4 + (m & 3), sl = (m >> 2) * 16 + (c & 15);
  float s1 = 0.f, sg = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {                         // fixed order: wave 0, 1, ..
    s1 += red[((size_t)q * NI4 + it) * 64 + sl];
    if (DUAL) sg += red[((size_t)q * NI4 + NTW * 4 + it) * 64 + sl];
  }
  gemm_epilogue<EPI, AT>(a, a.rows_live, m, n, s1, sg, pbias);
}

// The line: one row saves about 2 us of a 1600-wide chain and each further one gives 0.6 - 0.7 back, so the fourth breaks even there;
// narrower chains are still ahead with four.  At 8 rows the fused launch was 2 - 3 us slower at 1600 and 2048.  Wider rows (4096: 896 workgroups for FFN-up) lose already at one: 45.6 -> 48.4 us.
// Up to 512 columns, where four groups of threads share the rows, it is ahead or equal up to 16, and the chain has two launches less per
// layer for the host.  us per layer of such a chain, 7 launches / 5, as a graph and where the host needs 3.7 us per launch: 512 columns
// (RMS), 5 rows 19.7 / 17.1 and 28.4 / 23.9, 8 rows 19.9 / 17.6 and 29.1 / 24.2, 12 rows 20.1 / 18.9, 16 rows 20.2 / 20.4 and 27.7 / 25.8; float32,
// 512 columns, 8 rows 26.5 / 23.2, 16 rows 28.1 / 27.0; 256 columns, 16 rows 22.3 / 21.5.  (All rows in every thread: 8 rows 21.5 for 17.6.)
bool gemm_takes_norm(int d, int rows) { return rows <= 4 ? d <= 2048 : rows <= 16 && d <= 512; }

template <typename AT, int NTW, int EPI>
static void launch_gemm_norm_epi(const GemmArgs& a, const NormFusion& f, int rows, hipStream_t s) {
  const dim3 grid((a.n_tiles + NTW - 1) / NTW + (f.emb.rope ? 1 : 0));   // (one workgroup has them all)
  const int R = rows <= 4 ? rows : (rows + 3) / 4 * 4;    // (the kernel's, which strides LDS by it)
  const size_t lds = sizeof(AT) == 2 ? (size_t)R * a.K * 2 : (size_t)R * (a.K + 4) * 4;
#define SPRINTER_FUSED(R_) hipLaunchKernelGGL((k_gemm_norm<AT, R_, NTW, EPI>), grid, dim3(512), lds, s, a, f)
  if (rows == 1) SPRINTER_FUSED(1); else if (rows == 2) SPRINTER_FUSED(2); else if (rows == 3) SPRINTER_FUSED(3); else if (rows == 4) SPRINTER_FUSED(4);
  else if (rows <= 8) SPRINTER_FUSED(8); else if (rows <= 12) SPRINTER_FUSED(12); else SPRINTER_FUSED(16);
#undef SPRINTER_FUSED
}

void launch_gemm_norm(int dtype, int epi, const NormFusion& f, const void* W, const void* W2, int N, int K, const float* bias,
                      float* out_f32, int ldo, void* out_act, int out_K, int rows, hipStream_t s) {
  GemmArgs a;
  memset(&a, 0, sizeof a);
  a.W = W; a.W2 = W2; a.N = N; a.K = K; a.Kt = (K + 31) / 32; a.n_tiles = (N + 15) / 16;
  a.bias = bias; a.out_f32 = out_f32; a.ldo = ldo; a.out_act = out_act; a.out_K = out_K; a.rows_live = rows;
#define SPRINTER_EPI(AT, NTW)                                                                 \
  do {                                                                                        \
    if (epi == EPI_F32) launch_gemm_norm_epi<AT, NTW, EPI_F32>(a, f, rows, s);                \
    else if (epi == EPI_GELU) launch_gemm_norm_epi<AT, NTW, EPI_GELU>(a, f, rows, s);         \
    else launch_gemm_norm_epi<AT, NTW, EPI_SWIGLU>(a, f, rows, s);                            \
  } while (0)
  if (dtype == 0) SPRINTER_EPI(float, 1);
  else if (a.n_tiles >= 256 && a.Kt < 100) SPRINTER_EPI(bf16_t, 2);   // two column tiles per wave, as k_gemm16
  else SPRINTER_EPI(bf16_t, 1);
#undef SPRINTER_EPI
}

}  // namespace sprinter
