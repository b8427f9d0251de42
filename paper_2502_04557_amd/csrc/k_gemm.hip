// HIP kernels of the batched SPRINTER decode step for gfx950: the projection / FFN GEMMs
// (Alg. 2: the draft's and the target's forward passes).
#include "gemm.h"
#include <algorithm>
#include <cstring>

namespace sprinter {

// bf16-mode GEMM (float16 operands) on MFMA for at most 16 rows.  512 threads = 8 waves that split K; each wave owns NTW column tiles
// (16 columns each): D[m][n] += X[m][k] W[n][k].
// All 8 waves leave their partial sums in LDS and every thread then finishes ONE output element: it adds the 8
// partials in fixed order, applies bias / GELU / SwiGLU and stores.  With the element order chosen per
// output layout the 256 x NTW stores of the workgroup are contiguous: one 32-column operand tile for
// the activation outputs, 64-128 byte runs for float32 rows.  (When wave 0 alone ran the epilogue - 8 tanh and 16
// scattered 2-byte stores per lane for FFN-up - it took 2.2 of the kernel's 7.1 us.)
// Accumulator layout of v_mfma_f32_16x16x32: lane l, register v hold n = l % 16, m = (l / 16) * 4 + v.
template <int NTW, int EPI>
__global__ __launch_bounds__(512) void k_gemm16(GEMM_ARGS) {
  const GemmArgs a = gemm_args<EPI>(W_, X_, second_, Kt_, N_, rows_live_, ldo_, n_rows_, out_, more_);
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr bool ACT_OUT = (EPI == EPI_GELU || EPI == EPI_SWIGLU);
  constexpr int U = 4;      // k tiles per chunk and wave (8 and 16 measured slower)
  constexpr int NI = NTW * 4, NI2 = NI * (DUAL ? 2 : 1), NOUT = NTW * 256;
  __shared__ float red[8 * NI2 * 64];
  const int tid = threadIdx.x, lane = tid & 63, kw = wave_index();
  const int nt0 = blockIdx.x * NTW;
  const uint4* __restrict__ Wp = (const uint4*)a.W;
  const uint4* __restrict__ W2p = (const uint4*)a.W2;
  const uint4* __restrict__ Xp = (const uint4*)a.X;
  const int Kt = a.Kt;
  // Requests that depend on nothing are issued before the row count is even read: this wave's first weight
  // tiles and this thread's bias.
  uint4 wv[U][NTW], wv2[U][DUAL ? NTW : 1];
  auto load_weights = [&](int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int kc = min(kt + u * 8, Kt - 1);                     // clamped: always a valid tile
#pragma unroll
      for (int j = 0; j < NTW; ++j) {
        int nt = min(nt0 + j, a.n_tiles - 1);
        wv[u][j] = Wp[((size_t)nt * Kt + kc) * 64 + lane];
        if (DUAL) wv2[u][j] = W2p[((size_t)nt * Kt + kc) * 64 + lane];
      }
    }
  };
  // A lane holds 8 k of row lane % 16: lanes of rows the host knows not to exist skip their loads (a step with 3
  // rejected rows then pulls 3/16 of the activation bytes through the compute unit's memory pipeline, which carries
  // them next to the weight stream); what their registers hold only reaches output rows that are dropped.
  const bool row_live = (lane & 15) < a.rows_live;
  uint4 xv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) xv[u] = make_uint4(0u, 0u, 0u, 0u);
  auto load_x = [&](int kt) {                               // no dependence on the (device-side) row count
    if (row_live) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kc = min(kt + u * 8, Kt - 1);
        xv[u] = Xp[(size_t)kc * 64 + lane];
      }
    }
  };
  load_weights(min(kw, Kt - 1));
  load_x(min(kw, Kt - 1));
  // this thread's output element: (row m, column c of the workgroup's 16 NTW columns)
  int m, c;
  if (ACT_OUT) { m = (tid >> 3) & 15; c = (tid >> 7) * 8 + (tid & 7); }      // operand-tile order: 8 columns, 16 rows, next 8 columns
  else { m = tid / (16 * NTW); c = tid % (16 * NTW); }                      // row-major
  const int n = nt0 * 16 + c;
  const bool n_ok = tid < NOUT && n < a.N;
  const float pbias = (n_ok && a.bias) ? a.bias[n] : 0.f;
  int kv_b = 0, kv_slot = 0;
  if (EPI == EPI_QKV) { const int mc = min(m, a.rows_live - 1); kv_b = a.kv.b[mc]; kv_slot = a.kv.slot[mc]; }
  // (The row count is only needed by the epilogue: launches are sized by the host for rows that exist, so the loop
  // does not wait for it.)
  const int n_rows = *a.n_rows;
  f32x4 acc[NTW], acc2[DUAL ? NTW : 1];
#pragma unroll
  for (int j = 0; j < NTW; ++j) {
    acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (DUAL) acc2[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  }
  for (int kt = kw; kt < Kt; kt += 8 * U) {
    // Straight-line code: all loads of a chunk are issued together, k tiles beyond K are clamped on load and
    // zeroed as operands.  (A branch per k tile keeps the scheduler from hoisting the loads and serialises one
    // L2 latency per tile.)
    if (kt != kw) { load_weights(kt); load_x(kt); }         // (the first chunk is already on its way)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in_k = kt + u * 8 < Kt;
      const uint4 ah = in_k ? xv[u] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int j = 0; j < NTW; ++j) {
        acc[j] = mfma_f16(ah, wv[u][j], acc[j]);
        if (DUAL) {
          acc2[j] = mfma_f16(ah, wv2[u][j], acc2[j]);
        }
      }
    }
  }
  {
    float* dst = red + (size_t)kw * NI2 * 64;
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dst[(j * 4 + v) * 64 + lane] = acc[j][v];
        if (DUAL) dst[(NI + j * 4 + v) * 64 + lane] = acc2[j][v];
      }
  }
  __syncthreads();
  if (tid >= NOUT) return;
  const int it = (c >> 4) * 4 + (m & 3), sl = (m >> 2) * 16 + (c & 15);
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {                             // fixed order: wave 0, 1, ..
    s1 += red[((size_t)q * NI2 + it) * 64 + sl];
    if (DUAL) s2 += red[((size_t)q * NI2 + NI + it) * 64 + sl];
  }
  gemm_epilogue<EPI, bf16_t>(a, n_rows, m, n, s1, s2, pbias, kv_b, kv_slot);
}

// bf16-mode GEMM for 17 .. 64 rows (MT row tiles of 16) of outputs too narrow for k_gemm_tile, NTW column tiles per workgroup,
// K split over the 8 waves.  At these row counts a workgroup pulls the whole activation matrix (MT x 1 KiB per k tile,
// from L2) for 1 KiB of weights per k tile, so the kernel lives on memory-level parallelism: two register
// buffers, the loads of chunk c + 1 (weights and all MT row tiles) are in flight while the
// MFMAs of chunk c run, and there is no branch inside the loop.  Row tiles beyond the row count are
// computed on whatever the buffers hold and dropped by the epilogue; k tiles beyond K are clamped on load
// and their weight operand zeroed.
template <int MT, int NTW, int EPI>
__global__ __launch_bounds__(512) void k_gemm_rows(GEMM_ARGS) {
  const GemmArgs a = gemm_args<EPI>(W_, X_, second_, Kt_, N_, rows_live_, ldo_, n_rows_, out_, more_);
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr int NWT = NTW * (DUAL ? 2 : 1);          // weight tiles per k tile and wave
  constexpr int U = (MT * NWT >= 8) ? 1 : 2, STEP = 8 * U;   // k tiles per buffer
  constexpr int NI = MT * NWT * 4;
  __shared__ float red[4 * NI * 64];
  const int lane = threadIdx.x & 63, kw = wave_index();
  const int nt0 = blockIdx.x * NTW, Kt = a.Kt;
  const uint4* __restrict__ Wp = (const uint4*)a.W + lane;
  const uint4* __restrict__ W2p = DUAL ? (const uint4*)a.W2 + lane : nullptr;
  const uint4* __restrict__ Xp = (const uint4*)a.X + lane;
  size_t wrow[NTW];
#pragma unroll
  for (int j = 0; j < NTW; ++j) wrow[j] = (size_t)min(nt0 + j, a.n_tiles - 1) * Kt * 64;
  struct Buf { uint4 w[U][NWT], xh[U][MT]; };
  // (as in k_gemm16: a lane whose row exists in no launch - the host's bound - skips its activation loads; with 18
  // rows the second row tile costs an eighth of its bytes)
  bool row_live[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) row_live[mt] = mt * 16 + (lane & 15) < a.rows_live;
  auto load = [&](Buf& b, int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kc = min(kt + u * 8, Kt - 1);
#pragma unroll
      for (int j = 0; j < NTW; ++j) {
        b.w[u][j] = Wp[wrow[j] + (size_t)kc * 64];
        if (DUAL) b.w[u][NTW + j] = W2p[wrow[j] + (size_t)kc * 64];
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      if (row_live[mt]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int kc = min(kt + u * 8, Kt - 1);
          b.xh[u][mt] = Xp[((size_t)mt * Kt + kc) * 64];
        }
      }
    }
  };
  f32x4 acc[NWT][MT];
#pragma unroll
  for (int j = 0; j < NWT; ++j)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[j][mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const Buf& b, int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in_k = kt + u * 8 < Kt;
#pragma unroll
      for (int j = 0; j < NWT; ++j) {
        const uint4 w1 = in_k ? b.w[u][j] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          acc[j][mt] = mfma_f16(b.xh[u][mt], w1, acc[j][mt]);
        }
      }
    }
  };
  Buf A, B;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) A.xh[u][mt] = B.xh[u][mt] = make_uint4(0u, 0u, 0u, 0u);
  load(A, min(kw, Kt - 1));
  constexpr int NO = (MT * NTW + 1) / 2;                      // output elements per thread
  int kv_b[EPI == EPI_QKV ? NO : 1] = {0}, kv_slot[EPI == EPI_QKV ? NO : 1] = {0};
  if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int i = 0; i < NO; ++i) {
      const int mc = min((i * 512 + (int)threadIdx.x) / (16 * NTW), a.rows_live - 1);
      kv_b[i] = a.kv.b[mc]; kv_slot[i] = a.kv.slot[mc];
    }
  }
  const int n_rows = *a.n_rows;                               // only the epilogue needs it (passes are sized by the host)
  // (the scheduling barriers keep the compiler from sinking a buffer's loads down to their first use)
  for (int kt = kw; kt < Kt; kt += 2 * STEP) {
    load(B, kt + STEP);
    __builtin_amdgcn_sched_barrier(0);
    compute(A, kt);
    __builtin_amdgcn_sched_barrier(0);
    load(A, kt + 2 * STEP);
    __builtin_amdgcn_sched_barrier(0);
    compute(B, kt + STEP);
    __builtin_amdgcn_sched_barrier(0);
  }
  // the 8 partial accumulators are summed pairwise through LDS: (0+4, 1+5, 2+6, 3+7), (0+2, 1+3), (0+1)
#pragma unroll
  for (int half = 4; half >= 1; half >>= 1) {
    if (kw >= half && kw < 2 * half) {
      float* dst = red + (size_t)(kw - half) * NI * 64;
#pragma unroll
      for (int j = 0; j < NWT; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int v = 0; v < 4; ++v) dst[((j * MT + mt) * 4 + v) * 64 + lane] = acc[j][mt][v];
    }
    __syncthreads();
    if (kw < half) {
      const float* src = red + (size_t)kw * NI * 64;
#pragma unroll
      for (int j = 0; j < NWT; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[j][mt][v] += src[((j * MT + mt) * 4 + v) * 64 + lane];
    }
    __syncthreads();
  }
  // Wave 0 now holds the totals; it hands them to the whole workgroup through LDS and every thread finishes
  // MT * NTW / 2 (rounded up) output elements, in an order that makes the workgroup's stores contiguous per output layout
  // (one wave running the epilogue for up to 64 values per lane was a serial tail of several microseconds).
  if (kw == 0) {
#pragma unroll
    for (int j = 0; j < NWT; ++j)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((j * MT + mt) * 4 + v) * 64 + lane] = acc[j][mt][v];
  }
  __syncthreads();
  constexpr bool ACT_OUT = (EPI == EPI_GELU || EPI == EPI_SWIGLU);
#pragma unroll
  for (int i = 0; i < NO; ++i) {
    const int o = i * 512 + (int)threadIdx.x;        // element index among the MT*16 x NTW*16 outputs
    if (o >= 256 * MT * NTW) break;
    int mt, m16, c;
    if (ACT_OUT) {                                   // operand-tile order: 8 columns, 16 rows, next 8 columns, next row tile
      const int rest = o >> 7;
      m16 = (o >> 3) & 15; c = (rest % (2 * NTW)) * 8 + (o & 7); mt = rest / (2 * NTW);
    } else {                                         // row-major
      const int m_all = o / (16 * NTW);
      c = o % (16 * NTW); mt = m_all >> 4; m16 = m_all & 15;
    }
    const int j = c >> 4, n = nt0 * 16 + c, m = mt * 16 + m16;
    const int sl = (m16 >> 2) * 16 + (c & 15), v = m16 & 3;
    const float s1 = red[((j * MT + mt) * 4 + v) * 64 + sl];
    const float s2 = DUAL ? red[(((NTW + j) * MT + mt) * 4 + v) * 64 + sl] : 0.f;
    if (m >= n_rows || n >= a.N) continue;
    const float bias = a.bias ? a.bias[n] : 0.f;
    gemm_epilogue<EPI, bf16_t>(a, n_rows, m, n, s1, s2, bias, kv_b[EPI == EPI_QKV ? i : 0], kv_slot[EPI == EPI_QKV ? i : 0]);
  }
}

// bf16-mode GEMM for at most 16 rows whose output only has to exist as a sum: O-proj and FFN-down add into the
// residual stream, and the layer norm that follows reads the whole row anyway.  K is split into SK shares
// over workgroups (workgroup = NTW column tiles x one share), each share leaves its partial product in
// part[s] and the norm kernel adds residual + bias + the shares in fixed order.  No reduction step, no
// fences, and every workgroup reads only its share of the activations - which at 16 rows cost as much as
// the weights: a workgroup needs 64 B of activations (L2) per k for 32 B of weights per k and tile.
template <int NTW>
__global__ __launch_bounds__(512) void k_gemm16_part(const void* W_, const void* X_, int Kt_, int N_, int rows_live_, int shares_, float* part_, const int* n_rows_, size_t part_stride_) {
  GemmArgs a;
  a.W = W_; a.X = X_; a.Kt = Kt_; a.N = a.ldo = N_; a.n_tiles = (N_ + 15) >> 4; a.rows_live = rows_live_; a.SK = shares_; a.part = part_; a.n_rows = n_rows_; a.part_stride = part_stride_;
  constexpr int U = 4;
  __shared__ float red[8 * NTW * 4 * 64];
  const int lane = threadIdx.x & 63, kw = wave_index();
  const int n_groups = (a.n_tiles + NTW - 1) / NTW;
  const int g = blockIdx.x % n_groups, sk = blockIdx.x / n_groups;
  const int nt0 = g * NTW, Kt = a.Kt;
  const int k0 = (int)((long long)Kt * sk / a.SK), k1 = (int)((long long)Kt * (sk + 1) / a.SK);
  const uint4* __restrict__ Wp = (const uint4*)a.W;
  const uint4* __restrict__ Xp = (const uint4*)a.X;
  uint4 wv[U][NTW];
  auto load_weights = [&](int kt) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kc = min(kt + u * 8, k1 - 1);                // clamped: always a tile of this share
#pragma unroll
      for (int j = 0; j < NTW; ++j) wv[u][j] = Wp[((size_t)min(nt0 + j, a.n_tiles - 1) * Kt + kc) * 64 + lane];
    }
  };
  const bool row_live = (lane & 15) < a.rows_live;            // (as in k_gemm16: rows that exist in no launch are not fetched)
  uint4 xv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) xv[u] = make_uint4(0u, 0u, 0u, 0u);
  auto load_x = [&](int kt) {
    if (row_live) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int kc = min(kt + u * 8, k1 - 1);
        xv[u] = Xp[(size_t)kc * 64 + lane];
      }
    }
  };
  load_weights(min(k0 + kw, k1 - 1));
  load_x(min(k0 + kw, k1 - 1));
  const int n_rows = *a.n_rows;                               // only the stores need it
  f32x4 acc[NTW];
#pragma unroll
  for (int j = 0; j < NTW; ++j) acc[j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int kt = k0 + kw; kt < k1; kt += 8 * U) {
    if (kt != k0 + kw) { load_weights(kt); load_x(kt); }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in_k = kt + u * 8 < k1;
      const uint4 ah = in_k ? xv[u] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
      for (int j = 0; j < NTW; ++j) {
        acc[j] = mfma_f16(ah, wv[u][j], acc[j]);
      }
    }
  }
  {
    float* dst = red + (size_t)kw * NTW * 4 * 64;
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[(j * 4 + v) * 64 + lane] = acc[j][v];
  }
  __syncthreads();
  // one output element per thread, row-major: the 8 partial sums in fixed order, stores in 64-128 byte runs
  const int tid = threadIdx.x;
  if (tid >= NTW * 256) return;
  const int m = tid / (16 * NTW), c = tid % (16 * NTW), n = nt0 * 16 + c;
  const int it = (c >> 4) * 4 + (m & 3), sl = (m >> 2) * 16 + (c & 15);
  float sum = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) sum += red[((size_t)q * NTW * 4 + it) * 64 + sl];
  if (n < a.N && m < n_rows) (a.part + (size_t)sk * a.part_stride)[(size_t)m * a.ldo + n] = sum;
}

// float32 GEMM on the float32 matrix pipes (v_mfma_f32_16x16x4_f32: exact float32 products, float32 sums).  A workgroup
// owns 16 columns and MT row tiles of 16; its 8 waves split K.  Operands come straight from the row-major matrices: lane
// (l16, lq) takes four consecutive k of row / column l16 with one 16-byte load, and the four products of a load use
// k = 4 lq + 0 .. 3 in both operands, so 16 k cost one load per operand and four matrix instructions.  U groups of 16 k
// are requested together before the first product waits: at these widths (K <= 2048) that is one or two memory round trips
// per wave, which is what bounds the kernel - the vector version (one wave per column, 8 rows at a time, the row loads
// under a branch per row) paid one round trip per row and 256 k: 768 x 256 at 24 rows 15.8 -> 4.2 us; O-proj and FFN-down
// of a 512-wide model (K = 512 and 2048) at 6 - 32 rows 28 -> 4 - 6 us with K shares, at one row 7.2 -> 3.8 us.
// blockIdx.y = pass over 16 MT rows.
template <int MT, int U, int EPI>
__global__ __launch_bounds__(512) void k_gemm_f32(const void* W_, const void* X_, const void* second_, int K_, int N_, int rows_live_, int shares_, const int* n_rows_, void* out_, int ldo_, size_t part_stride_) {
  GemmArgs a;                                           // second: bias, or W2; out: EPI_PART: the shares' buffer
  a.W = W_; a.X = X_; a.W2 = second_; a.bias = EPI == EPI_SWIGLU ? nullptr : (const float*)second_; a.K = K_; a.N = N_; a.rows_live = rows_live_; a.n_rows = n_rows_;
  a.out_f32 = a.part = (float*)out_; a.out_act = out_; a.ldo = a.out_K = ldo_; a.part_stride = part_stride_;
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr int NA = DUAL ? 2 : 1;
  __shared__ float red[8][NA * MT * 4][64];
  const int tid = threadIdx.x, lane = tid & 63, kw = wave_index();
  const int l16 = lane & 15, lq = lane >> 4, K = a.K;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * MT * 16;
  // EPI_PART: blockIdx.z = K share, the partial product goes to part[share] (summed by the norm that follows)
  const int all_groups = (K + 15) >> 4, s0 = all_groups * (int)blockIdx.z / shares_;
  const int n_groups = all_groups * (int)(blockIdx.z + 1) / shares_ - s0;
  const int g0 = s0 + n_groups * kw / 8, g1 = s0 + n_groups * (kw + 1) / 8;
  const int n_col = min(n0 + l16, a.N - 1);             // columns beyond N are computed on the last one and dropped
  const float* __restrict__ wr = (const float*)a.W + (size_t)n_col * K;
  const float* __restrict__ wr2 = DUAL ? (const float*)a.W2 + (size_t)n_col * K : nullptr;
  const float* __restrict__ X = (const float*)a.X;
  bool live[MT];                                        // lanes of rows that do not exist load nothing and enter as zeros
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) live[mt] = m0 + mt * 16 + l16 < a.rows_live;
  // This thread's output element (consecutive threads: consecutive columns of a row); its bias and current value are
  // requested here, not after the sums.
  const int mr = tid >> 4, c = tid & 15, m_out = m0 + mr, n_out = n0 + c;
  const int n_rows = *a.n_rows;
  const bool out_ok = mr < MT * 16 && m_out < a.rows_live && n_out < a.N;
  const float pbias = (EPI != EPI_PART && out_ok && a.bias) ? a.bias[n_out] : 0.f;
  f32x4 acc[NA * MT];
#pragma unroll
  for (int i = 0; i < NA * MT; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
  for (int g = g0; g < g1; g += U) {
    float4 wv[U], wv2[DUAL ? U : 1], xv[U][MT];
#pragma unroll
    for (int u = 0; u < U; ++u) {                       // K is a multiple of 4; k beyond it is clamped here and zeroed below
      const int k = min(min(g + u, g1 - 1) * 16 + lq * 4, K - 4);
      wv[u] = *reinterpret_cast<const float4*>(wr + k);
      if (DUAL) wv2[u] = *reinterpret_cast<const float4*>(wr2 + k);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xv[u][mt] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (live[mt]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int k = min(min(g + u, g1 - 1) * 16 + lq * 4, K - 4);
          xv[u][mt] = *reinterpret_cast<const float4*>(X + (size_t)(m0 + mt * 16 + l16) * K + k);
        }
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool on = g + u < g1 && (g + u) * 16 + lq * 4 < K;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w1 = on ? (&wv[u].x)[e] : 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32((&xv[u][mt].x)[e], w1, acc[mt], 0, 0, 0);
        if (DUAL) {
          const float w2 = on ? (&wv2[u].x)[e] : 0.f;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[MT + mt] = __builtin_amdgcn_mfma_f32_16x16x4f32((&xv[u][mt].x)[e], w2, acc[MT + mt], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NA * MT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[kw][i * 4 + v][lane] = acc[i][v];
  __syncthreads();
  if (!out_ok) return;
  const int mt = mr >> 4, sl = ((mr & 15) >> 2) * 16 + c;
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {                         // fixed order: wave 0, 1, ..
    s1 += red[q][mt * 4 + (mr & 3)][sl];
    if (DUAL) s2 += red[q][(MT + mt) * 4 + (mr & 3)][sl];
  }
  if (m_out >= n_rows) return;
  if constexpr (EPI == EPI_PART) (a.part + (size_t)blockIdx.z * a.part_stride)[(size_t)m_out * a.ldo + n_out] = s1;
  else gemm_epilogue<EPI, float>(a, n_rows, m_out, n_out, s1, s2, pbias);
}

template <int EPI>
static void launch_gemm_f32(const GemmArgs& a, int max_rows, int shares, hipStream_t s) {
  // two row tiles per pass from 17 rows on; as many groups of 16 k per request as a wave's share of K has, at most 8
  const int per_wave = ((a.K + 15) / 16 + 8 * shares - 1) / (8 * shares), mt = max_rows <= 16 ? 1 : 2;
  const dim3 grid(a.n_tiles, (max_rows + 16 * mt - 1) / (16 * mt), shares);
#define SPRINTER_F32(MT_, U_) hipLaunchKernelGGL((k_gemm_f32<MT_, U_, EPI>), grid, dim3(512), 0, s, a.W, a.X, EPI == EPI_SWIGLU ? a.W2 : (const void*)a.bias, a.K, a.N, a.rows_live, shares, a.n_rows, \
    EPI == EPI_PART ? (void*)a.part : EPI == EPI_F32 ? (void*)a.out_f32 : a.out_act, EPI == EPI_PART || EPI == EPI_F32 ? a.ldo : a.out_K, a.part_stride)
  if (mt == 1) { if (per_wave <= 2) SPRINTER_F32(1, 2); else if (per_wave <= 4) SPRINTER_F32(1, 4); else SPRINTER_F32(1, 8); }
  else { if (per_wave <= 2) SPRINTER_F32(2, 2); else if (per_wave <= 4) SPRINTER_F32(2, 4); else SPRINTER_F32(2, 8); }
#undef SPRINTER_F32
}

template <int EPI>
static void launch_gemm_bf16(const GemmArgs& a, int max_rows, hipStream_t s) {
  // Up to 16 rows: one 16-column tile per workgroup (two per wave for wide outputs), K split over its 8 waves.
  // (Fewer rows of narrower models have the norm inside: k_gemm_norm.hip.  Measured and dropped: splitting K over workgroups with a last-arriver reduction - its two device-scope fences
  // cost more than the 4 us they save; a variant that requests all of a wave's weight and activation
  // tiles up front (K <= 2048) - no faster.)
  // wide outputs with a short K: two column tiles per wave share the activation fragments (at K = 4096 one tile per
  // workgroup is faster: QKV 12288x4096 26 against 32 us, FFN-up 2x11008x4096 40 against 48 us)
  if (max_rows <= 16 && a.n_tiles >= 256 && a.Kt < 100)
    hipLaunchKernelGGL((k_gemm16<2, EPI>), dim3((a.n_tiles + 1) / 2), dim3(512), 0, s, GEMM_VALUES(a, EPI));
  else if (max_rows <= 16) hipLaunchKernelGGL((k_gemm16<1, EPI>), dim3(a.n_tiles), dim3(512), 0, s, GEMM_VALUES(a, EPI));
  else if (gemm_takes_tile(EPI, a.N, max_rows)) launch_gemm_tile(EPI, a, max_rows, 1, s);
  else {
    // 17 .. 64 rows.  Two column tiles per wave, which share the activation fragments, where one would need a second round of
    // workgroups (one per compute unit): 4352 x 4096 (272 tiles) at 20 / 40 / 64 rows 15.8 / 19.1 / 23.3 us with one, 12.6 / 14.9 /
    // 17.6 with two; 4096 x 4096 (256) 10.0 / 12.1 / 14.5 and 12.6 / 14.9 / 17.5.
    constexpr bool DUAL = EPI == EPI_SWIGLU;
#define SPRINTER_ROWS(MT_, NTW_) hipLaunchKernelGGL((k_gemm_rows<MT_, NTW_, EPI>), grid, dim3(512), 0, s, GEMM_VALUES(a, EPI))
    const int mt = (max_rows + 15) / 16, ntw = !DUAL && a.n_tiles > 256 ? 2 : 1;
    const dim3 grid((a.n_tiles + ntw - 1) / ntw);
    if constexpr (!DUAL) {
      if (ntw == 2) { if (mt == 2) SPRINTER_ROWS(2, 2); else if (mt == 3) SPRINTER_ROWS(3, 2); else SPRINTER_ROWS(4, 2); }
    }
    if (ntw == 1) { if (mt == 2) SPRINTER_ROWS(2, 1); else if (mt == 3) SPRINTER_ROWS(3, 1); else SPRINTER_ROWS(4, 1); }
#undef SPRINTER_ROWS
  }
}

void launch_gemm(int dtype, int epi, const void* W, const void* W2, const void* X, size_t x_elems, const int* n_rows,
                 int N, int K, const float* bias, float* out_f32, int ldo, void* out_act, int out_K,
                 int max_rows, hipStream_t s) {
  GemmArgs a;
  memset(&a, 0, sizeof a);
  a.x_elems = x_elems;
  a.W = W; a.W2 = W2; a.X = X; a.n_rows = n_rows; a.N = N; a.K = K;
  a.Kt = (K + 31) / 32; a.n_tiles = (N + 15) / 16;
  a.bias = bias; a.out_f32 = out_f32; a.ldo = ldo; a.out_act = out_act; a.out_K = out_K; a.rows_live = max_rows;
  if (dtype == 0) {
    switch (epi) {
      case EPI_F32: launch_gemm_f32<EPI_F32>(a, max_rows, 1, s); break;
      case EPI_GELU: launch_gemm_f32<EPI_GELU>(a, max_rows, 1, s); break;
      default: launch_gemm_f32<EPI_SWIGLU>(a, max_rows, 1, s); break;
    }
  } else {
    switch (epi) {
      case EPI_F32: launch_gemm_bf16<EPI_F32>(a, max_rows, s); break;
      case EPI_GELU: launch_gemm_bf16<EPI_GELU>(a, max_rows, s); break;
      default: launch_gemm_bf16<EPI_SWIGLU>(a, max_rows, s); break;
    }
  }
}

void launch_gemm_qkv(const void* W, const void* X, size_t x_elems, const int* n_rows, int N, int K, const float* bias, float* y,
                     const KvDest& kv, int max_rows, hipStream_t s) {
  GemmArgs a;
  memset(&a, 0, sizeof a);
  a.W = W; a.X = X; a.x_elems = x_elems; a.n_rows = n_rows; a.N = N; a.K = K; a.Kt = (K + 31) / 32; a.n_tiles = (N + 15) / 16;
  a.bias = bias; a.out_f32 = y; a.ldo = N; a.kv = kv; a.rows_live = max_rows;
  launch_gemm_bf16<EPI_QKV>(a, max_rows, s);
}

int launch_gemm_part(int dtype, const void* W, const void* X, size_t x_elems, const int* n_rows, int N, int K, float* part,
                     size_t part_stride, int max_shares, const float* bias, float* h, int max_rows, hipStream_t s) {
  GemmArgs a;
  memset(&a, 0, sizeof a);
  a.W = W; a.X = X; a.x_elems = x_elems; a.n_rows = n_rows; a.N = N; a.K = K;
  a.Kt = (K + 31) / 32; a.n_tiles = (N + 15) / 16; a.ldo = N;
  a.part = part; a.part_stride = part_stride; a.rows_live = max_rows;
  if (dtype == 0) {
    // shares of at least 32 groups of 16 k (4 per wave: one round of requests), at most 4 (the norm's smaller variant)
    const int sk = std::max(1, std::min(std::min(4, max_shares), (K + 15) / 16 / 32));
    launch_gemm_f32<EPI_PART>(a, max_rows, sk, s);
    return sk;
  }
  if (max_rows <= 16) {
    // shares: fill the 256 compute units, at least 12 k tiles per share; long K takes two column tiles per wave.  us per layer, FFN-down with one / two: 1088 x 4352, 16 rows 31.7 /
    // 32.3; 2048 x 5504 45.3 / 46.2; 1600 x 6400 39.5 / 39.3; 2560 x 10240, 8 rows 61.2 / 57.9; 5120 x 13824 164.5 / 160.7; 5120 x 20480 162.4 / 154.8; 8192 x 32768, 16 rows 369.2 / 357.8.
    const bool two = a.Kt >= 192 && a.n_tiles >= 64;
    const int groups = two ? (a.n_tiles + 1) / 2 : a.n_tiles;
    int sk = std::min(4, 256 / groups);              // (4: the norm kernel's smaller partial-sum variant)
    if (sk > max_shares) sk = max_shares;
    while (sk > 1 && a.Kt / sk < 12) --sk;
    if (sk < 1) sk = 1;
    a.SK = sk;
    if (two) hipLaunchKernelGGL((k_gemm16_part<2>), dim3(groups * sk), dim3(512), 0, s, a.W, a.X, a.Kt, a.N, a.rows_live, a.SK, a.part, a.n_rows, a.part_stride);
    else hipLaunchKernelGGL((k_gemm16_part<1>), dim3(groups * sk), dim3(512), 0, s, a.W, a.X, a.Kt, a.N, a.rows_live, a.SK, a.part, a.n_rows, a.part_stride);
    return sk;
  }
  a.bias = bias; a.out_f32 = h;
  return launch_gemm_tile(EPI_PART, a, max_rows, max_shares, s);
}

}  // namespace sprinter
