// HIP kernels of the batched SPRINTER decode step for gfx950: the layer of a pass of few rows in five launches.  O-projection and FFN-down add
// themselves to the residual rows and leave the statistics of what they wrote (k_gemm_resid); QKV projection and FFN-up normalise
// those rows for themselves (k_norm_gemm).
#include "gemm.h"
#include <algorithm>
#include <cstring>
#include <type_traits>

namespace sprinter {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Workgroup barrier that orders LDS traffic only: __syncthreads() also waits for the weights in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// A buffer of n bytes: loads beyond it give zeros and fetch nothing.
__device__ __forceinline__ auto bytes_at(const void* p, int n) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, n, 0x00020000); }
__device__ __forceinline__ float last_lane(float v) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 63)); }

// Statistics of the residual rows: for every row and every `cols` consecutive columns {sum, sum of squared distances from their mean}
// (RMS norm: {-, sum of squares}), as the workgroup that wrote the columns took them.  A row's mean and variance are put together from them
// with no pass over the row: variance d = sum over the groups of theirs + cols (group mean - mean)^2, the update of Chan, Golub and LeVeque,
// which loses nothing against two passes.

// Column groups of the statistics: 16 / split columns each, at most 256 groups where a product reads them.  float32 rows hold their k side by side, so four columns
// fill lines too: 512 x 2048, 1 row 5.0 -> 4.0 us, 8 rows 6.0 -> 5.4 but the norms behind it lose that again.  From 2049 columns on 16 stay ahead, also
// where nobody reads the statistics: us per layer with 16 / 8 columns per workgroup, 2112 columns, 8 / 16 / 32 rows 47.3 / 52.6 / 65.8, 49.5 / 58.4 / 73.1; 3072 69.2 / 78.7 / 92.3, 72.9 / 84.6 / 103.6.
static __host__ __device__ constexpr int resid_split(bool bf16, int N, int rows) { return N > 2048 ? 1 : !bf16 && N <= 1024 && rows <= 4 ? 4 : 2; }

// What k_norm_gemm takes: rows per thread RT and groups of threads RG, 8 columns a thread; RT = 0: no kernel.  The rule of gemm_takes_norm is this one, so that no
// row count is taken that a kernel does not hold.
struct NormShape { int rt, rg; };
static constexpr NormShape norm_shape(bool bf16, int d, int rows) {
  const int rg = d <= 512 ? 8 : d <= 1024 ? 4 : d <= 2048 ? 2 : 1, most = d > (bf16 ? 4096 : 2048) ? 0 : bf16 && rg < 8 ? 4 : 2;
  int rt = 1;
  while (rt * rg < rows) rt *= 2;
  return {rt <= most ? rt : 0, rg};
}
static __host__ __device__ constexpr int norm_stat_loads(bool bf16, int rg) { return bf16 ? (rg >= 2 ? 8 / rg : 4) : rg == 8 ? 2 : 4; }   // of 64 column groups, for a row's statistics
static constexpr bool norm_shapes_hold() {
  for (int bf16 = 0; bf16 < 2; ++bf16)
    for (int d = 64; d <= 8192; d += 64)
      for (int rows = 1; rows <= 40; ++rows) {
        const NormShape f = norm_shape(bf16, d, rows);
        if (f.rt && (f.rt * f.rg < rows || f.rt * f.rg > 16 || 512 / f.rg * 8 < d || d / 16 * resid_split(bf16, d, rows) > 64 * norm_stat_loads(bf16, f.rg))) return false;
      }
  return true;
}
static_assert(norm_shapes_hold(), "rows, columns or statistics that a kernel does not hold");

// A chain of short dependent launches is what a pass of few rows is, and the norm as a launch of its own two of a layer's seven: 3 - 4 us for a few KiB of
// work.  Every workgroup of the product that follows can normalise the rows for itself, if that is cheap: here it reads them once, in one piece, with
// at most 256 groups of statistics, and the weights it needs are requested behind them and arrive meanwhile.  (Before, it read residual rows and
// up to four partial products, took the statistics in two passes through LDS and four barriers that waited for all weights in flight: 0.5 us a row
// of 1600 columns, paid after the weights had arrived.)  The code is straight: buffers whose bounds make loads beyond them zeros instead of
// branches, so that every wait counts the loads behind the one it is for; a barrier waits for LDS only.
// A layer in a chain (graph over all layers, cold weights), us, before -> with these two kernels -> and their arguments preloaded: 1600 columns (25 heads, 6400), 1 row
// 28.0 -> 25.8 -> 24.6, 4 rows 34.3 -> 28.3 -> 27.0, 8 rows (seven launches before) 34.2 -> 30.6 -> 29.4; 768 (3072), 1 row 18.4 -> 16.3 -> 15.3, 16 rows (seven) 25.6 ->
// 23.0 -> 22.4; 2048 (gate + up 8192), 1 row 39.0 -> 35.3 -> 34.0, 4 rows 42.3 -> 36.5 -> 36.0; 4096 (11008; seven), 3 rows 95.3 -> 84.3 -> 82.1; 4096 (14336; seven), 1 row 97.2 ->
// 87.5 -> 85.6; 512 (1344), 4 rows 20.0 -> 17.4, 16 rows 21.6 -> 20.0; float32, 512 (2048), 1 row 22.1 -> 19.3 -> 18.3, 8 rows 24.7 -> 22.8 -> 22.0.
// What bounds it: the weights at 4 - 5 TB/s and, of 5.4 us at 15 MB, the start of a dependent launch, 1.6 us.
// R = RT RG rows: RG groups of 512 / RG threads, a thread takes 8 columns of RT rows.  U: units of K in flight per wave.
struct RowSource { EmbedSource emb; float* h_out; };    // EMB: the rows are embeddings; workgroup 0 starts the residual stream with them
// second: the norm's offset b, or W2.  d / 16 * resid_split groups of statistics.
template <typename AT, int ARCH, int RT, int RG, int NTW, int EPI, bool EMB>
__global__ __launch_bounds__(512) void k_norm_gemm(const float* h, const float* stat, const float* g, const void* second, const void* W, int d, int rows, int N, float eps,
                                                   void* out, const float* bias, std::conditional_t<EMB, RowSource, Nothing> from) {
  constexpr bool BF = sizeof(AT) == 2;
  constexpr bool DUAL = EPI == EPI_SWIGLU, ACT_OUT = BF && EPI != EPI_F32;
  constexpr int R = RT * RG, CG = 512 / RG, WR = 8 / RG, NW = NTW * (DUAL ? 2 : 1), NI4 = NW * 4, SR = (R + 7) / 8;
  constexpr int U = (BF ? 1 : 2) * 16 / RG > 8 ? 8 : (BF ? 1 : 2) * 16 / RG, NG = norm_stat_loads(BF, RG);   // units in flight; loads of a row's statistics
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float2 s_stat[R];
  __shared__ float s_part[2][R][WR];
  __shared__ float red[8 * NI4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), l16 = lane & 15, lq = lane >> 4;
  const int nt0 = blockIdx.x * NTW, n_tiles = (N + 15) >> 4, split = resid_split(BF, d, rows), groups = d / 16 * split, units = BF ? d >> 5 : d >> 4;
  if constexpr (EMB && ARCH == 1) {
    if (__builtin_expect(nt0 >= n_tiles, 0)) {        // one workgroup more for the rows' rotary factors
      const int half = from.emb.dh >> 1;
      for (int i = tid; i < rows * half; i += 512) rope_factors(from.emb, i / half, i % half);
      return;
    }
  }
  const float cols = 16 / split, inv_cols = split / 16.f;                     // (a power of two)
  // ---- statistics, residual rows, gain and offset; then the weights
  float2 st[SR][NG];
  if constexpr (!EMB) {
#pragma unroll
    for (int j = 0; j < SR; ++j) if (w + 8 * j < rows) {   // (scalar; the first loads, so no later wait depends on it)
      const float2* sp = (const float2*)stat + (size_t)min(w + 8 * j, rows - 1) * groups;
#pragma unroll
      for (int i = 0; i < NG; ++i) st[j][i] = sp[min(lane + 64 * i, groups - 1)];
    }
  }
  const int col = tid % CG, rg = w / WR, n_ch = d >> 3, c8 = min(col, n_ch - 1) * 8;
  const bool mine = col < n_ch;
  float x[RT][8], gg[8], bb[8];
  if constexpr (EMB) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int r = min(rg * RT + i, rows - 1);
      const int tok = min(max(from.emb.rd.tok[r], 0), from.emb.V - 1), pos = max(from.emb.rd.pos[r], 0);
      load_row((const AT*)from.emb.tok_emb + (size_t)tok * d + c8, x[i]);
      if (from.emb.pos_emb) {
        float p[8];
        load_row((const AT*)from.emb.pos_emb + (size_t)min(pos, from.emb.max_pos - 1) * d + c8, p);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[i][e] += p[e];
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < RT; ++i) load_row(h + (size_t)min(rg * RT + i, rows - 1) * d + c8, x[i]);
  }
  load_row(g + c8, gg);
  if (ARCH == 0) load_row((const float*)second + c8, bb);
  __builtin_amdgcn_sched_barrier(0);
  const unsigned w_lane = BF ? lane * 16 : (l16 * d + lq * 4) * 4;
  auto tile = [&](int j) {
    const int nt = nt0 + j % NTW;
    const char* m = (const char*)(DUAL && j >= NTW ? second : W);
    return bytes_at(m + (size_t)nt * 16 * d * sizeof(AT), nt < n_tiles ? (BF ? 16 : min(16, N - nt * 16)) * d * (int)sizeof(AT) : 0);
  };
  u32x4 wv[U][NW];
  auto load_unit = [&](int u, int unit) {
#pragma unroll
    for (int j = 0; j < NW; ++j) wv[u][j] = __builtin_amdgcn_raw_buffer_load_b128(tile(j), unit_offset(BF || unit < units, w_lane, unit, BF ? 1024 : 64), 0, 0);
  };
#pragma unroll
  for (int u = 0; u < U; ++u) load_unit(u, w + 8 * u);
  int m, c;                                             // this thread's output element, as in k_gemm16
  if (ACT_OUT) { m = (tid >> 3) & 15; c = (tid >> 7) * 8 + (tid & 7); }
  else { m = tid / (16 * NTW); c = tid % (16 * NTW); }
  const int n = nt0 * 16 + c;
  const bool out_ok = tid < NTW * 256 && m < rows && n < N;
  const float pbias = (out_ok && bias) ? bias[n] : 0.f;
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (EMB) {
    if (blockIdx.x == 0 && mine) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
        if (rg * RT + i < rows) {
          float4* o = reinterpret_cast<float4*>(from.h_out + (size_t)(rg * RT + i) * d + c8);
          o[0] = make_float4(x[i][0], x[i][1], x[i][2], x[i][3]);
          o[1] = make_float4(x[i][4], x[i][5], x[i][6], x[i][7]);
        }
    }
    float part[RT], mean[RT];
    auto totals = [&](int slot) {
#pragma unroll
      for (int i = 0; i < RT; ++i) part[i] = wave_total(mine ? part[i] : 0.f);
      if (lane == 63) {
#pragma unroll
        for (int i = 0; i < RT; ++i) s_part[slot][rg * RT + i][w % WR] = part[i];
      }
      lds_barrier();
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        part[i] = 0.f;
#pragma unroll
        for (int q = 0; q < WR; ++q) part[i] += s_part[slot][rg * RT + i][q];
      }
    };
#pragma unroll
    for (int i = 0; i < RT; ++i) mean[i] = 0.f;
    if (ARCH == 0) {
#pragma unroll
      for (int i = 0; i < RT; ++i) part[i] = ((x[i][0] + x[i][1]) + (x[i][2] + x[i][3])) + ((x[i][4] + x[i][5]) + (x[i][6] + x[i][7]));
      totals(0);
#pragma unroll
      for (int i = 0; i < RT; ++i) mean[i] = part[i] / (float)d;
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      part[i] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float t = x[i][e] - mean[i]; part[i] += t * t; }
    }
    totals(1);
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < RT; ++i) s_stat[rg * RT + i] = make_float2(mean[i], 1.0f / sqrtf(part[i] / (float)d + eps));
    }
  } else {
#pragma unroll
    for (int j = 0; j < SR; ++j) {
      float mean = 0.f, s = 0.f;
      if (ARCH == 0) {
#pragma unroll
        for (int i = 0; i < NG; ++i) s += lane + 64 * i < groups ? st[j][i].x : 0.f;
        mean = last_lane(wave_total(s)) / (float)d;
        s = 0.f;
      }
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        float q = st[j][i].y;
        if (ARCH == 0) { const float t = st[j][i].x * inv_cols - mean; q += cols * (t * t); }
        s += lane + 64 * i < groups ? q : 0.f;
      }
      const float rstd = 1.0f / sqrtf(last_lane(wave_total(s)) / (float)d + eps);
      if (lane == 0 && w + 8 * j < R) s_stat[w + 8 * j] = make_float2(mean, rstd);
    }
  }
  lds_barrier();
  // ---- normalised rows to LDS: float16 operand slots [k / 8][row] of 16 bytes, or float32 rows (4 floats of padding)
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int r = rg * RT + i;
    const float2 ms = s_stat[r];
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      o[e] = (x[i][e] - ms.x) * ms.y * gg[e];
      if (ARCH == 0) o[e] += bb[e];
    }
    if (mine) {
      if constexpr (BF) *reinterpret_cast<uint4*>(smem + ((size_t)col * R + r) * 16) = make_uint4(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]), pk_f16(o[4], o[5]), pk_f16(o[6], o[7]));
      else {
        float4* p = reinterpret_cast<float4*>(smem + ((size_t)r * (d + 4) + c8) * 4);
        p[0] = make_float4(o[0], o[1], o[2], o[3]);
        p[1] = make_float4(o[4], o[5], o[6], o[7]);
      }
    }
  }
  lds_barrier();
  // ---- product: wave w takes units (32 k, or 16 in float32) w, w + 8, ..
  const int xrow = min(l16, R - 1);                     // (outputs of rows that do not exist are dropped)
  f32x4 acc[NW];
#pragma unroll
  for (int j = 0; j < NW; ++j) acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  auto use = [&](int u, int unit) {
    const int k = min(unit, units - 1);                 // (beyond: zero weights)
    if constexpr (BF) {
      const uint4 xv = *reinterpret_cast<const uint4*>(smem + ((size_t)(k * 4 + lq) * R + xrow) * 16);
#pragma unroll
      for (int j = 0; j < NW; ++j) acc[j] = mfma_f16(xv, make_uint4(wv[u][j].x, wv[u][j].y, wv[u][j].z, wv[u][j].w), acc[j]);
    } else {
      const float4 xv = *reinterpret_cast<const float4*>(smem + ((size_t)xrow * (d + 4) + k * 16 + lq * 4) * 4);
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.x, __uint_as_float(wv[u][j].x), acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.y, __uint_as_float(wv[u][j].y), acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.z, __uint_as_float(wv[u][j].z), acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv.w, __uint_as_float(wv[u][j].w), acc[j], 0, 0, 0);
      }
    }
  };
  int unit = w;
  for (; unit + 8 * U < units; unit += 8 * U) {         // (scalar)
#pragma unroll
    for (int u = 0; u < U; ++u) { use(u, unit + 8 * u); load_unit(u, unit + 8 * (U + u)); }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) use(u, unit + 8 * u);
#pragma unroll
  for (int j = 0; j < NW; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((size_t)w * NI4 + j * 4 + v) * 64 + lane] = acc[j][v];
  __syncthreads();
  if (!out_ok) return;
  const int it = (c >> 4) * 4 + (m & 3), sl = (m >> 2) * 16 + (c & 15);
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {                         // fixed order: wave 0, 1, ..
    s1 += red[((size_t)q * NI4 + it) * 64 + sl];
    if (DUAL) s2 += red[((size_t)q * NI4 + NTW * 4 + it) * 64 + sl];
  }
  if constexpr (EPI == EPI_F32) ((float*)out)[(size_t)m * N + n] = s1 + pbias;
  else if constexpr (EPI == EPI_GELU) act_store<AT>((AT*)out, m, n, N, gelu_tanh(s1 + pbias));
  else act_store<AT>((AT*)out, m, n, N, silu(s1) * s2);
}

template <int C>
__device__ __forceinline__ float columns_sum(float v) {   // over C = 4, 8 or 16 consecutive lanes
  if constexpr (C > 4) return group_sum<C>(v);
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));           // quad_perm [1,0,3,2]
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));     // quad_perm [2,3,0,1]
}
// O-projection and FFN-down of at most 16 rows, some of at most 32 (gemm_takes_norm, gemm_adds_rows): h += bias + X W^T in place, and the statistics of what was written.  A workgroup has all of K for its columns, so
// that it can finish them, and 16 / S columns instead of 16 where that takes to fill the chip (N <= 2048): a weight load then carries S k
// tiles of the columns - 128 bytes of each for S = 2, a line -, as many bytes per workgroup as K in S shares.  What that costs is the activations of
// all of K in every workgroup, and the address unit takes 16 cycles per load whatever it brings: so where an operand's 16 rows are not all there, a load
// carries 16 / RP tiles of RP rows side by side.  Products of unequal k tiles land in accumulator elements of their own and are dropped at the end.
// Four accumulators at least, and the 8 waves' sums in pairs: what K in shares over workgroups won in precision stays (error of the residual rows against 64 bits,
// 2-norm, K in shares -> in order -> so: 1600 x 6400, 4 rows 8.7e-8 -> 9.5e-8 -> 6.9e-8; 4096 x 14336, 16 rows 1.58e-7 -> 2.13e-7 -> 1.19e-7).
// us, K in shares over workgroups and the sum left to the norm -> this: 1600 x 6400, 4 rows 6.3 -> 6.7, 16 rows 7.1 -> 9.0; 1600 x 1600 3.8 -> 3.8;
// 4096 x 14336 and 4096 x 4096 at 5 - 16 rows 24.7 -> 22.5 and 12.1 -> 8.1; the norms behind it 3.4 -> 2.9, or gone (above).
// RP: rows an activation load carries (4, 8 or 16); MT: operands of 16 rows.  UG: groups of T = max(16 / RP, S) k tiles in flight per wave.
template <typename AT, int ARCH, int S, int RP, int UG, int MT>
__global__ __launch_bounds__(512) void k_gemm_resid(const void* W, const void* X, int K, int rows, float* h, const float* bias, float* stat, int N) {
  constexpr bool BF = sizeof(AT) == 2;
  constexpr int C = 16 / S, P = 16 / RP, T = P > S ? P : S, NX = T / P, NWL = T / S, NM = NX > NWL ? NX : NWL, KU = BF ? 32 : 16;
  constexpr int NA = P >= S ? P / S : S;                // accumulators: which of their elements are sums of matching k is below
  constexpr int D = NA < 4 ? 4 / NA : 1;                // each D times, for groups in turn
  static_assert(MT == 1 || (BF && RP == 16), "");
  static_assert(P >= S || P == 1, "an accumulator for every tile s of a column, as they are matched below");
  __shared__ float red[8 * MT * 4 * 64];
  const int tid = threadIdx.x, lane = tid & 63, w = wave_index(), l16 = lane & 15, lq = lane >> 4;
  const int kt = (K + KU - 1) / KU, groups = (kt + T - 1) / T, n0 = blockIdx.x * C;
  const int ws = l16 / C, wc = l16 % C, xp = l16 / RP, xr = l16 % RP;
  const auto rw = BF ? bytes_at((const char*)W + (size_t)(n0 >> 4) * kt * 1024, kt * 1024) : bytes_at((const char*)W + (size_t)n0 * K * 4, C * K * 4);
  const auto rx = BF ? bytes_at(X, MT * kt * 1024) : bytes_at(X, rows * K * 4);
  const unsigned w_lane = BF ? ws * 1024 + (lq * 16 + (n0 & 15) + wc) * 16 : wc * K * 4 + (ws * 16 + lq * 4) * 4;
  const unsigned x_lane = xr < rows ? (BF ? xp * 1024 + (lq * 16 + xr) * 16 : xr * K * 4 + (xp * 16 + lq * 4) * 4) : NOWHERE;
  constexpr int TB = BF ? 1024 : 64;                    // bytes from one k tile to the next
  u32x4 wv[UG][NWL], xv[UG][NX][MT];
  auto load_group = [&](int u, int g) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int t = g * T + i * P;
      // (beyond K zeros on both sides; with several operands the buffer goes on there: other rows, whose infinities must not meet a zero weight)
      xv[u][i][0] = __builtin_amdgcn_raw_buffer_load_b128(rx, unit_offset(BF ? MT == 1 || t < kt : (t + xp) * KU + lq * 4 < K, x_lane, t, TB), 0, 0);
#pragma unroll
      for (int j = 1; j < MT; ++j)                      // (the next 16 rows are an operand tile row further)
        xv[u][i][j] = __builtin_amdgcn_raw_buffer_load_b128(rx, unit_offset(t < kt && 16 * j + l16 < rows, lane * 16, j * kt + t, 1024), 0, 0);
    }
#pragma unroll
    for (int i = 0; i < NWL; ++i) {
      const int t = g * T + i * S;
      wv[u][i] = __builtin_amdgcn_raw_buffer_load_b128(rw, unit_offset(BF || (t + ws) * KU + lq * 4 < K, w_lane, t, TB), 0, 0);
    }
  };
#pragma unroll
  for (int u = 0; u < UG; ++u) load_group(u, w + 8 * u);
  // this thread's output elements: a row's columns in consecutive lanes
  constexpr int OUT = (MT * RP * C + 511) / 512;
  float res[OUT];
#pragma unroll
  for (int o = 0; o < OUT; ++o) {
    const int m = (o * 512 + tid) / C, n = n0 + tid % C;
    res[o] = 0.f;
    if (m < rows) { res[o] = h[(size_t)m * N + n]; if (bias) res[o] += bias[n]; }
  }
  f32x4 acc[MT][NA][D];
#pragma unroll
  for (int j = 0; j < MT; ++j)
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
      for (int v = 0; v < D; ++v) acc[j][i][v] = (f32x4){0.f, 0.f, 0.f, 0.f};
  auto use = [&](int u) {
#pragma unroll
    for (int i = 0; i < NM; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const u32x4 x = xv[u][i % NX][j], wt = wv[u][i % NWL];
        f32x4& sum = acc[j][i % NA][u % D];
        if constexpr (BF) sum = mfma_f16(make_uint4(x.x, x.y, x.z, x.w), make_uint4(wt.x, wt.y, wt.z, wt.w), sum);
        else {
#pragma unroll
          for (int e = 0; e < 4; ++e) sum = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x[e]), __uint_as_float(wt[e]), sum, 0, 0, 0);
        }
      }
  };
  int g = w;
  for (; g + 8 * UG < groups; g += 8 * UG) {            // (scalar)
#pragma unroll
    for (int u = 0; u < UG; ++u) { use(u); load_group(u, g + 8 * (UG + u)); }
  }
#pragma unroll
  for (int u = 0; u < UG; ++u) use(u);
  // Operand row RP p + r is row r at k tile p of a load, operand column C s + c column c at tile s: accumulator i sums matching tiles
  // where p = S i + s (P >= S), or s = i (P = 1).
  const int mine = P >= S ? (lq * 4 / RP) / S : ws;
#pragma unroll
  for (int j = 0; j < MT; ++j) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      if constexpr (D == 2) acc[j][i][0] += acc[j][i][1];
      if constexpr (D == 4) acc[j][i][0] = (acc[j][i][0] + acc[j][i][1]) + (acc[j][i][2] + acc[j][i][3]);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float x = acc[j][0][0][v];
#pragma unroll
      for (int i = 1; i < NA; ++i) x = mine == i ? acc[j][i][0][v] : x;
      red[((w * MT + j) * 4 + v) * 64 + lane] = x;
    }
  }
  __syncthreads();
#pragma unroll
  for (int o = 0; o < OUT; ++o) {
    const int m = (o * 512 + tid) / C, c = tid % C, n = n0 + c;
    if (m >= MT * RP) return;
    float sum[8 * T];
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int row = (P == 1 ? 0 : t * RP) + (m & (RP - 1)), s = t % S;
        sum[q * T + t] = red[((q * MT + m / RP) * 4 + (row & 3)) * 64 + (row >> 2) * 16 + s * C + c];
      }
#pragma unroll
    for (int half = 4 * T; half; half >>= 1)            // in pairs, always the same ones
#pragma unroll
      for (int i = 0; i < half; ++i) sum[i] += sum[i + half];
    const float v = res[o] + sum[0];
    float mean = 0.f, dv = v, s1 = 0.f;
    if (ARCH == 0) { s1 = columns_sum<C>(v); mean = s1 * (1.0f / C); dv = v - mean; }
    const float s2 = columns_sum<C>(dv * dv);
    if (m >= rows) return;
    h[(size_t)m * N + n] = v;
    if (stat && c == 0) reinterpret_cast<float2*>(stat)[(size_t)m * (N / C) + blockIdx.x] = make_float2(s1, s2);
  }
}

// The line: us per layer, seven launches / five.  1600 columns: 8 rows 34.2 / 30.6, 10 rows 35.9 / 35.7, 16 rows 38.4 / 38.9; 2048 (gate + up): 8 rows 43.6 / 38.6, 10 rows 44.1 / 44.6;
// 4096: 4 rows 96.5 / 85.3, 5 rows 92.9 / 96.8; 768: 16 rows 25.6 / 23.4; 1024: 16 rows 28.8 / 27.2.  (Activations of more than 8 rows fill an operand; 5 rows of 4096 in
// every thread leave one workgroup per compute unit.)  float32 rows take twice the LDS: seven / five launches, 256 columns, 16 rows
// 26.0 / 23.0, 512 30.8 / 27.8; 1024, 8 rows 40.0 / 35.5 (gate + up 40.5 / 37.5); 1536, 4 rows 65.4 / 53.5; 2048 72.6 / 67.0.  bf16, 2112 - 3584 columns, 4 rows: 46.6 / 45.5 to 85.0 / 79.1.
bool gemm_takes_norm(int dtype, int d, int rows) { return norm_shape(dtype != 0, d, rows).rt != 0; }
// Whether a product of K adds itself to the residual rows although the norm behind it is a launch.  Its workgroups have all of K, and one of them fills a compute unit: what decides
// is how many of those the last round of 16 columns per workgroup leaves idle, where K in shares would fill them, and how much K there is.  us per layer of a target pass of 4 to 16
// layers, K in shares / added (O-projection and FFN-down changed one at a time; two runs of one side differ by 0.3 %):
// - O-projection (K = d).  2112 columns, 8 / 16 / 32 rows 45.8 / 50.0 / 62.3 -> 45.2 / 49.1 / 61.2; 3072, 8 / 32 rows 73.0 / 88.7 -> 72.0 / 89.0; 4096, 17 rows 118.7 -> 117.7; 5120,
//   4 / 16 / 24 rows 147.0 / 174.9 / 174.7 -> 144.9 / 173.7 / 178.4; 6144, 4 / 8 / 16 rows 197.8 / 206.1 / 227.4 -> 197.6 / 207.3 / 227.3; 8192, 8 / 16 / 24 rows 332.6 / 357.7 / 368.6 ->
//   330.5 / 357.2 / 370.0.  17 - 32 rows of at most 2048 columns: 576 - 2048 columns 2 - 6 % ahead (1600, 17 / 32 rows 46.7 / 50.3 -> 44.8 / 48.8).
// - FFN-down (K = 2.7 d - 4 d).  Up to 8 rows where the last round is 7/8 full: 2112, 8 rows 45.2 -> 46.6; 2560 57.7 -> 59.4; 3072 72.0 -> 71.9; 3584 86.4 -> 85.9; 3840 93.5 -> 92.0; 4096
//   (14336) 117.4 -> 116.4; 5120, 4 / 8 rows 144.9 / 154.6 -> 149.2 / 157.4; 6144 207.3 -> 212.4; 8192 330.5 -> 326.9.  Beyond, only in one round that is full: 12 / 24 rows of 3584
//   95.2 / 100.3 -> 96.8 / 102.4; 3840 102.1 / 107.8 -> 103.0 / 109.8; 4096 109.5 / 120.1 -> 109.4 / 118.2 (28 - 32 rows 1 % behind); 8192 347.1 / 370.0 -> 349.9 / 376.5; 5120, 24 rows 178.4 -> 194.6.
// - K of at most 2048: 17 - 32 rows, FFN-down of 768 (2048), 24 rows 32.4 -> 32.0, of 640 (1728) 30.4 -> 29.8; 1600 columns, 6400 of K 12.6 -> 13.1; 256 columns 6.2 -> 6.3.
bool gemm_adds_rows(int dtype, int d, int K, int rows) {
  if (dtype == 0 || d <= 512 || rows > 32 || K > FEW_ROWS_MAX_K) return false;
  if (K <= 2048) return d > 2048 || rows > 16;
  if (d <= 2048) return false;
  if (2 * K <= 3 * d) return rows <= (d <= 4096 ? 32 : d <= 5120 ? 16 : 8);
  const int wgs = d / 16, idle = -wgs & 255;
  return rows <= (wgs <= 256 && idle <= 4 ? 32 : 8 * idle <= wgs + idle ? 8 : 0);
}

struct NormGemmArgs { const float *h, *stat, *g; const void *second, *W; const float* bias; void* out; int d, N, n_tiles, rows; float eps; RowSource from; };

template <typename AT, int ARCH, int NTW, int EPI, bool EMB>
static bool launch_norm_gemm_rows(const NormGemmArgs& a, hipStream_t s) {
  std::conditional_t<EMB, RowSource, Nothing> from;
  if constexpr (EMB) from = a.from;
  constexpr bool BF = sizeof(AT) == 2;
  const dim3 grid((a.n_tiles + NTW - 1) / NTW + (EMB && ARCH == 1 ? 1 : 0));
  const NormShape f = norm_shape(BF, a.d, a.rows);
#define SPRINTER_NG(RT, RG)                                                                                  \
  if (f.rt == RT && f.rg == RG) {                                                                            \
    const size_t lds = BF ? (size_t)RT * RG * a.d * 2 : (size_t)RT * RG * (a.d + 4) * 4;                        \
    hipLaunchKernelGGL((k_norm_gemm<AT, ARCH, RT, RG, NTW, EPI, EMB>), grid, dim3(512), lds, s, a.h, a.stat, a.g, a.second, a.W, a.d, a.rows, a.N, a.eps, a.out, a.bias, from);           \
    return true;                                                                                             \
  }
  if constexpr (NTW == 1) {
    SPRINTER_NG(1, 8) SPRINTER_NG(2, 8) SPRINTER_NG(1, 4) SPRINTER_NG(2, 4)
    if constexpr (BF) { SPRINTER_NG(4, 4) SPRINTER_NG(1, 1) SPRINTER_NG(2, 1) SPRINTER_NG(4, 1) }
  }
  SPRINTER_NG(1, 2) SPRINTER_NG(2, 2)
  if constexpr (BF) SPRINTER_NG(4, 2)
#undef SPRINTER_NG
  return false;
}

template <typename AT, int ARCH>
static bool launch_norm_gemm_arch(int epi, bool emb, const NormGemmArgs& a, hipStream_t s) {
  constexpr int ACT = ARCH == 0 ? EPI_GELU : EPI_SWIGLU;
  if constexpr (sizeof(AT) == 2) {
    if (a.n_tiles >= 256 && a.d > 1024 && a.d <= 2048) {   // two column tiles per wave, as k_gemm16
      if (epi != EPI_F32) return launch_norm_gemm_rows<AT, ARCH, 2, ACT, false>(a, s);
      return emb ? launch_norm_gemm_rows<AT, ARCH, 2, EPI_F32, true>(a, s) : launch_norm_gemm_rows<AT, ARCH, 2, EPI_F32, false>(a, s);
    }
  }
  if (epi != EPI_F32) return launch_norm_gemm_rows<AT, ARCH, 1, ACT, false>(a, s);
  return emb ? launch_norm_gemm_rows<AT, ARCH, 1, EPI_F32, true>(a, s) : launch_norm_gemm_rows<AT, ARCH, 1, EPI_F32, false>(a, s);
}

bool launch_norm_gemm(int dtype, int arch, int epi, const float* h, const float* stat, const float* g, const float* b, float eps, const EmbedSource* emb,
                      float* h_out, const void* W, const void* W2, int N, int d, const float* bias, void* out, int rows, hipStream_t s) {
  NormGemmArgs a;
  memset(&a, 0, sizeof a);
  a.h = h; a.stat = stat; a.g = g; a.second = arch == 0 ? (const void*)b : W2; a.W = W; a.bias = bias; a.out = out;   // (an offset and two matrices: no architecture has both)
  a.d = d; a.N = N; a.n_tiles = (N + 15) / 16; a.rows = rows; a.eps = eps;
  a.from.h_out = h_out;
  if (emb) a.from.emb = *emb;
  if (dtype == 0) return arch == 0 ? launch_norm_gemm_arch<float, 0>(epi, emb, a, s) : launch_norm_gemm_arch<float, 1>(epi, emb, a, s);
  return arch == 0 ? launch_norm_gemm_arch<bf16_t, 0>(epi, emb, a, s) : launch_norm_gemm_arch<bf16_t, 1>(epi, emb, a, s);
}

struct ResidArgs { const void *W, *X; float *h, *stat; const float* bias; int N, K, rows; };
template <typename AT, int ARCH, int S, int RP>
static void launch_gemm_resid_rows(const ResidArgs& a, hipStream_t s) {
  constexpr int T = 16 / RP > S ? 16 / RP : S, KU = sizeof(AT) == 2 ? 32 : 16;
#define SPRINTER_RES(UG) hipLaunchKernelGGL((k_gemm_resid<AT, ARCH, S, RP, UG, 1>), dim3(a.N * S / 16), dim3(512), 0, s, a.W, a.X, a.K, a.rows, a.h, a.bias, a.stat, a.N)
  // (up to 8 weight loads of 16 bytes per lane in flight; 16 where two of them make a group)
  if constexpr (T / S == 4) SPRINTER_RES(2);
  else {
    const int per_wave = ((a.K + KU - 1) / KU + 8 * T - 1) / (8 * T);
    if (per_wave <= 2) SPRINTER_RES(2); else if (per_wave <= 4) SPRINTER_RES(4); else SPRINTER_RES(8);
  }
#undef SPRINTER_RES
}
template <typename AT, int ARCH, int S>
static bool launch_gemm_resid_split(const ResidArgs& a, hipStream_t s) {
  if (a.rows <= 4) launch_gemm_resid_rows<AT, ARCH, S, 4>(a, s);
  else if (S == 4 || a.rows > 16) return false;
  else if constexpr (S <= 2) { if (a.rows <= 8) launch_gemm_resid_rows<AT, ARCH, S, 8>(a, s); else launch_gemm_resid_rows<AT, ARCH, S, 16>(a, s); }
  return true;
}
template <typename AT, int ARCH>
static bool launch_gemm_resid_arch(const ResidArgs& a, hipStream_t s) {
  const int S = resid_split(sizeof(AT) == 2, a.N, a.rows);
  if constexpr (sizeof(AT) == 2) {
#define SPRINTER_RES(S_) hipLaunchKernelGGL((k_gemm_resid<AT, ARCH, S_, 16, S_ == 1 ? 8 : 4, 2>), dim3(a.N * S_ / 16), dim3(512), 0, s, a.W, a.X, a.K, a.rows, a.h, a.bias, a.stat, a.N)
    if (a.rows > 16 && a.rows <= 32) { if (S == 1) SPRINTER_RES(1); else SPRINTER_RES(2); return true; }
#undef SPRINTER_RES
    return S == 1 ? launch_gemm_resid_split<AT, ARCH, 1>(a, s) : launch_gemm_resid_split<AT, ARCH, 2>(a, s);
  }
  else return S == 4 ? launch_gemm_resid_split<AT, ARCH, 4>(a, s) : S == 2 && launch_gemm_resid_split<AT, ARCH, 2>(a, s);
}
bool launch_gemm_resid(int dtype, int arch, const void* W, const void* X, int N, int K, const float* bias, float* h, float* stat, int rows, hipStream_t s) {
  if (K > FEW_ROWS_MAX_K) return false;
  const ResidArgs a{W, X, h, stat, bias, N, K, rows};
  if (dtype == 0) return arch == 0 ? launch_gemm_resid_arch<float, 0>(a, s) : launch_gemm_resid_arch<float, 1>(a, s);
  return arch == 0 ? launch_gemm_resid_arch<bf16_t, 0>(a, s) : launch_gemm_resid_arch<bf16_t, 1>(a, s);
}

}  // namespace sprinter
