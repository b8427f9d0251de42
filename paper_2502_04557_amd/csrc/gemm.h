// What the GEMM kernels (k_gemm.hip, k_gemm_norm.hip, k_gemm_tile.hip) share: launch arguments and the epilogue of one output
// element.
#pragma once
#include "dev.h"

namespace sprinter {

// =================================================================== GEMM
struct GemmArgs {
  const void* W; const void* W2; const void* X; const int* n_rows;
  int N, K, Kt, n_tiles;
  const float* bias; float* out_f32; int ldo; void* out_act; int out_K;
  size_t x_elems;     // elements the activation buffer X holds (bf16 mode)
  int SK; float* part; size_t part_stride;   // k_gemm16_part: K shares, partial outputs [SK][rows][N], floats per share
  int rows_live;      // the host's bound on the row count: rows from here on exist in no launch, their activations are not fetched
};

// bias: the column's bias (0 if none)
template <int EPI, typename AT>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int n_rows, int m, int n, float v, float v2, float bias) {
  if (m >= n_rows || n >= a.N) return;
  if (EPI == EPI_F32) a.out_f32[(size_t)m * a.ldo + n] = v + bias;
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
