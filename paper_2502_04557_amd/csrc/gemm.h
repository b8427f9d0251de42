// What the GEMM kernels (k_gemm.hip, k_gemm_norm.hip, k_gemm_tile.hip) share: launch arguments and the epilogue of one output
// element.
#pragma once
#include "dev.h"
#include <type_traits>

namespace sprinter {

// =================================================================== GEMM
struct GemmArgs {
  const void* W; const void* W2; const void* X; const int* n_rows;
  int N, K, Kt, n_tiles;
  const float* bias; float* out_f32; int ldo; void* out_act; int out_K;
  size_t x_elems;     // elements the activation buffer X holds (bf16 mode)
  int SK; float* part; size_t part_stride;   // k_gemm16_part: K shares, partial outputs [SK][rows][N], floats per share
  KvDest kv;          // EPI_QKV
  int rows_live;      // the host's bound on the row count: rows from here on exist in no launch, their activations are not fetched
};

// As arguments of k_gemm16 and k_gemm_rows.  second: bias, or W2 (gate + up has no bias).
template <int EPI> struct GemmMoreOf { using type = Nothing; };      // (named by the number: a kernel's signature must not name an enumerator of an unnamed type)
template <> struct GemmMoreOf<EPI_QKV> { using type = KvDest; };
template <int EPI> using GemmMore = typename GemmMoreOf<EPI>::type;
#define GEMM_ARGS const void *W_, const void *X_, const void *second_, int Kt_, int N_, int rows_live_, int ldo_, const int *n_rows_, void *out_, GemmMore<EPI> more_
#define GEMM_VALUES(a, EPI) (a).W, (a).X, EPI == EPI_SWIGLU ? (a).W2 : (const void*)(a).bias, (a).Kt, (a).N, (a).rows_live, \
    EPI == EPI_F32 || EPI == EPI_QKV ? (a).ldo : (a).out_K, (a).n_rows, EPI == EPI_F32 || EPI == EPI_QKV ? (void*)(a).out_f32 : (a).out_act, gemm_more<EPI>(a)
template <int EPI> inline GemmMore<EPI> gemm_more(const GemmArgs& a) { if constexpr (EPI == EPI_QKV) return a.kv; else return Nothing{}; }
template <int EPI>
__device__ __forceinline__ GemmArgs gemm_args(GEMM_ARGS) {
  GemmArgs a;
  a.W = W_; a.X = X_; a.W2 = second_; a.bias = EPI == EPI_SWIGLU ? nullptr : (const float*)second_; a.Kt = Kt_; a.N = N_; a.n_tiles = (N_ + 15) >> 4;
  a.rows_live = rows_live_; a.ldo = a.out_K = ldo_; a.n_rows = n_rows_; a.out_f32 = (float*)out_; a.out_act = out_;
  if constexpr (EPI == EPI_QKV) a.kv = more_;
  return a;
}

// EPI_QKV takes the place of the append launch of short passes (4.1 us per layer at 24 - 80 entries of 25 heads of 64; the product itself is
// not measurably slower for it): column n >= q_cols of an entry whose cache slot is (b, slot): its key or value element.  The values are bf16 bits.
__device__ __forceinline__ bf16_t* kv_element(const KvDest& d, int b, int slot, int n) {
  const bool v = n >= d.q_cols + d.kv_cols;
  const int c = n - d.q_cols - (v ? d.kv_cols : 0), head = c >> (d.dh == 128 ? 7 : 6), i = c & (d.dh - 1);   // (heads of 64 or 128)
  const size_t row = ((size_t)b * d.KVH + head) * (size_t)d.S * d.dh;
  return v ? (bf16_t*)d.vcache + row + vt_index(slot, i, d.dh) : (bf16_t*)d.kcache + row + (size_t)slot * d.dh + i;
}

// bias: the column's bias (0 if none); b, slot: EPI_QKV
template <int EPI, typename AT>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int n_rows, int m, int n, float v, float v2, float bias, int b = 0, int slot = 0) {
  if (m >= n_rows || n >= a.N) return;
  if (EPI == EPI_F32 || (EPI == EPI_QKV && n < a.kv.q_cols)) a.out_f32[(size_t)m * a.ldo + n] = v + bias;
  else if (EPI == EPI_QKV) *kv_element(a.kv, b, slot, n) = f2bf(v + bias);
  else if (EPI == EPI_GELU) act_store<AT>((AT*)a.out_act, m, n, a.out_K, gelu_tanh(v + bias));
  else act_store<AT>((AT*)a.out_act, m, n, a.out_K, silu(v) * v2);
}

// The kernel for 17 and more rows (k_gemm_tile.hip): whether a shape takes it, and its launch (returns the K shares of EPI_PART; 0: one
// share, added to a.out_f32).
// gemm_tile_choice: 16 x tile (0 - 4: 256 x 256, 128 x 128, 64 x 128, 64 x 64, 32 x 64) + K shares; a host function.
bool gemm_takes_tile(int epi, int N, int rows);
int gemm_tile_choice(int epi, int rows, int N, int K, int max_shares);
int launch_gemm_tile(int epi, const GemmArgs& a, int rows, int max_shares, hipStream_t s);

}  // namespace sprinter
