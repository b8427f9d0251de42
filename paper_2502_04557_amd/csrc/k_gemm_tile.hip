// HIP kernel of the batched SPRINTER decode step for gfx950: the GEMMs of many rows (prefill chunks, long work lists,
// large batches).
#include "gemm.h"
#include <algorithm>
#include <cstring>

namespace sprinter {

// bf16-mode GEMM (float16 operands) over a TM x TN output tile, both operands staged in LDS.  Weights and activations are
// stored as operand tiles of 16 rows x 32 k (1 KiB, in the lane order of the matrix instruction), so a tile goes from
// memory to LDS with one global_load_lds of 16 bytes a lane - no registers, no address swizzle - and from LDS into the
// instruction with one conflict-free ds_read_b128.  A ring of S stages of one k tile: at the top of k tile kt the wave waits
// until its own loads of stage kt + 1 have landed (its later ones stay in flight), the barrier makes that true for every
// wave and says that nobody reads stage kt - 1 any more, whose slot takes the loads of stage kt + S - 1.  The fragments of
// kt + 1 are read into a second register set between the matrix instructions of kt.
// The weight fragment is the first operand, so that the accumulator holds four consecutive COLUMNS of one row per lane:
// the epilogue stores 16 bytes of float32 or 8 bytes of an activation operand tile at a time.
// What bounds it (4096 rows, 256 x 256 tile): 1247 cycles per k tile, of which the matrix instructions are 1024 and the
// LDS (96 KiB of fragment reads and 32 KiB of arriving loads at 128 B a cycle) as many; the clock falls to 1.75 GHz under
// that load.  FFN-up 2 x 14336 x 4096: 856 -> 720 us (1.34 PFLOP/s), FFN-down 4096 x 11008: 327 -> 275, QKV 12288 x 4096:
// 458 -> 350, against one that shared only the activations through LDS and waited for all its loads at every barrier.
// Also measured: 32 x 32 x 16 instructions (8 - 20 % slower), a fifth stage (no faster), 4 waves of 128 x 128 (the compiler
// moves accumulators between register files: 1.5 times slower).
template <int WM, int WN, int MT, int NT, int S>
struct GemmTile {                                       // WM x WN waves, MT x NT operand tiles per wave, S stages
  static constexpr int wm = WM, wn = WN, mt = MT, nt = NT, stages = S, waves = WM * WN;
};
using TileL = GemmTile<4, 2, 4, 8, 4>;                  // 256 x 256, 128 KiB: one workgroup per compute unit
using TileM = GemmTile<2, 2, 4, 4, 5>;                  // 128 x 128, 80 KiB: two
using TileS = GemmTile<2, 2, 2, 4, 6>;                  // 64 x 128, 72 KiB: two

template <typename T, int EPI>
__global__ __launch_bounds__(T::waves * 64, 2) void k_gemm_tile(GemmArgs a, int x_tiles, int gm, int gn) {
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr int WN = T::wn, MT = T::mt, NT = T::nt, S = T::stages;
  constexpr int TMT = T::wm * MT, TNT = WN * NT, LT = TMT + TNT, PER = LT / T::waves;   // operand tiles per stage, per wave
  constexpr int COLS = DUAL ? NT / 2 : NT;              // output column tiles of a wave (SwiGLU: gate tiles, then up tiles)
  static_assert(LT % T::waves == 0 && NT % 2 == 0 && S >= 4, "");
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __shared__ u32x4 ring[S][LT][64];
  const int lane = threadIdx.x & 63, w = wave_index(), wm = w / WN, wn = w % WN;
  const int Kt = a.Kt;
  // EPI_PART: blockIdx.y = K share, the partial product goes to part[share] (summed by the norm that follows)
  const int sk = (EPI == EPI_PART) ? blockIdx.y : 0, SK = (EPI == EPI_PART) ? gridDim.y : 1;
  const int k0 = (int)((long long)Kt * sk / SK), k1 = (int)((long long)Kt * (sk + 1) / SK);
  // Workgroups go round-robin over the 8 XCDs: each XCD takes a contiguous run of tiles, ordered in bands of GM row groups,
  // so that what it has in flight at a time (32 compute units) shares rows and columns in its own L2.
  constexpr int GM = TMT >= 16 ? 4 : 8;
  const int n_blk = gm * gn, id = blockIdx.x, xcd = id & 7, q = n_blk >> 3, rem = n_blk & 7;
  const int t = xcd * q + min(xcd, rem) + (id >> 3);
  const int band = t / (GM * gn), in_band = t - band * GM * gn, bh = min(GM, gm - band * GM);
  const int bm = band * GM + in_band % bh, bn = in_band / bh;
  // this wave's PER operand tiles of a stage; tiles beyond the buffers are clamped, their products dropped by the epilogue
  const char* src[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int l = w * PER + i;
    const void* base;
    int tile;
    if (l < TMT) {
      base = a.X;
      tile = min(bm * TMT + l, x_tiles - 1);
    } else {
      const int j = l - TMT, jw = j / NT, jj = j % NT;
      const bool up = DUAL && jj >= COLS;
      base = up ? a.W2 : a.W;
      tile = min((bn * WN + jw) * COLS + (up ? jj - COLS : jj), a.n_tiles - 1);
    }
    src[i] = (const char*)base + (size_t)tile * Kt * 1024 + lane * 16;
  }
  auto issue = [&](int kt) {                            // (k tiles beyond the share: its last one again, never read)
    const size_t off = (size_t)min(kt, k1 - 1) * 1024;
    const int slot = (kt - k0) % S;
#pragma unroll
    for (int i = 0; i < PER; ++i)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[i] + off),
                                       (__attribute__((address_space(3))) void*)&ring[slot][w * PER + i][0], 16, 0, 0);
  };
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  struct Frag { u32x4 x[MT], w[NT]; };
  auto read = [&](Frag& f, int kt) {
    const u32x4* s = &ring[(kt - k0) % S][0][lane];
#pragma unroll
    for (int j = 0; j < NT; ++j) f.w[j] = s[(TMT + wn * NT + j) * 64];
#pragma unroll
    for (int i = 0; i < MT; ++i) f.x[i] = s[(wm * MT + i) * 64];
  };
  auto mul = [&](const Frag& f) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[i][j] = mfma_f16(__builtin_bit_cast(uint4, f.w[j]), __builtin_bit_cast(uint4, f.x[i]), acc[i][j]);
  };
  auto top = [&](int kt) {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((S - 3) * PER) : "memory");
    issue(kt + S - 1);
    __builtin_amdgcn_sched_barrier(0);
  };
  // fragment reads of the next k tile between the matrix instructions of this one (left alone, the scheduler sinks the
  // reads to the end of the block)
  auto weave = [&]() {
    constexpr int PACE = MT * NT >= 2 * (MT + NT) ? 2 : 1;
#pragma unroll
    for (int i = 0; i < MT + NT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, PACE, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, MT * NT, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < S - 1; ++i) issue(k0 + i);
  const int n_rows = *a.n_rows;                         // only the epilogue needs it
  Frag A, B;
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((S - 2) * PER) : "memory");
  __builtin_amdgcn_sched_barrier(0);
  read(A, k0);
  int kt = k0;
  for (; kt + 2 <= k1; kt += 2) {
    top(kt);
    read(B, kt + 1);
    mul(A);
    weave();
    top(kt + 1);
    read(A, kt + 2);
    mul(B);
    weave();
  }
  if (kt < k1) mul(A);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the clamped loads of the last stages still write to LDS
  // lane (lq, l16): row l16 of a row tile, columns 4 lq .. + 3 of a column tile (N is a multiple of 8)
  const int l16 = lane & 15, lq = lane >> 4;
  float* part = (EPI == EPI_PART) ? a.part + (size_t)sk * a.part_stride : nullptr;
#pragma unroll
  for (int j = 0; j < COLS; ++j) {
    const int n = ((bn * WN + wn) * COLS + j) * 16 + lq * 4;
    if (n >= a.N) continue;
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if (EPI != EPI_PART && a.bias) bias = *reinterpret_cast<const float4*>(a.bias + n);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = (bm * TMT + wm * MT + i) * 16 + l16;
      if (m >= n_rows) continue;
      const f32x4 c = acc[i][j];
      if constexpr (EPI == EPI_PART) {
        *reinterpret_cast<float4*>(part + (size_t)m * a.ldo + n) = make_float4(c[0], c[1], c[2], c[3]);
      } else if constexpr (EPI == EPI_F32) {
        *reinterpret_cast<float4*>(a.out_f32 + (size_t)m * a.ldo + n) =
            make_float4(c[0] + bias.x, c[1] + bias.y, c[2] + bias.z, c[3] + bias.w);
      } else {
        float o[4];
        if constexpr (EPI == EPI_GELU) {
          o[0] = gelu_tanh(c[0] + bias.x); o[1] = gelu_tanh(c[1] + bias.y);
          o[2] = gelu_tanh(c[2] + bias.z); o[3] = gelu_tanh(c[3] + bias.w);
        } else {
          const f32x4 u = acc[i][COLS + j];
#pragma unroll
          for (int v = 0; v < 4; ++v) o[v] = silu(c[v]) * u[v];
        }
        *reinterpret_cast<uint2*>((bf16_t*)a.out_act + act_idx<bf16_t>(m, n, a.out_K)) = make_uint2(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]));
      }
    }
  }
}

// Which tile, and how many K shares (partial products), for a shape: the one with the smallest estimate of
//   max(rounds of workgroups x cycles of a workgroup, padded products / rate) + the shares' way through memory,
// with the measured cycles per k tile of a workgroup that has its compute unit for itself / shares it with another, and the
// rate (PFLOP/s) that the tile reaches on a full chip.  Over 60 shapes of 100 - 4096 rows (K 768 - 14336, N 768 - 14336) the
// pick is within 10 % of the best of the three tiles and 1 / 2 / 4 / 8 shares, in 50 of them within 4 %.
struct TileCost { int tm, tn, per_cu; float alone, shared, rate; };
static float tile_us(const TileCost& c, int rows, int N, int Kt, bool dual, int sk) {
  const int cols = c.tn / (dual ? 2 : 1), slots = 256 * c.per_cu;
  const int wgs = (rows + c.tm - 1) / c.tm * ((N + cols - 1) / cols) * sk;
  const float kt = (float)Kt / sk, start = 5500.f;      // cycles before the first product and after the last
  const int full = wgs / slots, rest = wgs % slots;
  const float cycles = full * (start + c.shared * kt) + (rest > 256 ? start + c.shared * kt : rest > 0 ? start + c.alone * kt : 0.f);
  return std::max(cycles / 2400.f, 2.f * wgs * c.tm * c.tn * kt * 32 / c.rate * 1e-9f);
}

template <int EPI>
static int launch_tile_epi(GemmArgs a, int rows, int max_shares, hipStream_t s) {
  constexpr bool DUAL = EPI == EPI_SWIGLU;
  static const TileCost cost[3] = {{256, 256, 1, 1247.f, 1247.f, 1.33f}, {128, 128, 2, 530.f, 800.f, 1.16f}, {64, 128, 2, 340.f, 520.f, 0.92f}};
  int best = 0, sk = 1;
  float best_us = 1e30f;
  for (int i = 0; i < 3; ++i)
    for (int k = 1; k <= max_shares && (k == 1 || a.Kt / k >= 8); ++k) {
      // a share is written once and read once by the norm: 4.5 TB/s each way, half of the write hidden
      const float us = tile_us(cost[i], rows, a.N, a.Kt, DUAL, k) + (EPI == EPI_PART ? 1.5f * rows * a.N * 4.f * k / 4.5e6f : 0.f);
      if (us < best_us) { best_us = us; best = i; sk = k; }
    }
  const int x_tiles = (int)(a.x_elems / ((size_t)a.Kt * 512));
  const int gm = (rows + cost[best].tm - 1) / cost[best].tm, cols = cost[best].tn / (DUAL ? 2 : 1), gn = (a.N + cols - 1) / cols;
  const dim3 grid(gm * gn, sk);
  if (best == 0) hipLaunchKernelGGL((k_gemm_tile<TileL, EPI>), grid, dim3(TileL::waves * 64), 0, s, a, x_tiles, gm, gn);
  else if (best == 1) hipLaunchKernelGGL((k_gemm_tile<TileM, EPI>), grid, dim3(TileM::waves * 64), 0, s, a, x_tiles, gm, gn);
  else hipLaunchKernelGGL((k_gemm_tile<TileS, EPI>), grid, dim3(TileS::waves * 64), 0, s, a, x_tiles, gm, gn);
  return sk;
}

// Under 128 workgroups of the smallest tile the K-split kernels of k_gemm.hip, which put every column tile in a workgroup of
// its own, are ahead: QKV 6144 x 4096 at 128 rows (96 workgroups) 20.6 against 24.3 us, 3072 x 2048 at 256 rows (96) 13.3
// against 14.6; 6144 x 4096 at 200 rows (192) 29.7 against 26.3, 12288 x 4096 at 100 rows (192) 35.7 against 26.4.
bool gemm_takes_tile(int epi, const GemmArgs& a, int rows, int max_shares) {
  if (rows < 97) return false;
  const int cols = epi == EPI_SWIGLU ? 64 : 128, shares = epi == EPI_PART ? std::max(1, std::min(max_shares, a.Kt / 8)) : 1;
  return (rows + 63) / 64 * ((a.N + cols - 1) / cols) * shares >= 128;
}

int launch_gemm_tile(int epi, const GemmArgs& a, int rows, int max_shares, hipStream_t s) {
  switch (epi) {
    case EPI_F32: return launch_tile_epi<EPI_F32>(a, rows, 1, s);
    case EPI_GELU: return launch_tile_epi<EPI_GELU>(a, rows, 1, s);
    case EPI_SWIGLU: return launch_tile_epi<EPI_SWIGLU>(a, rows, 1, s);
    default: return launch_tile_epi<EPI_PART>(a, rows, max_shares, s);
  }
}

}  // namespace sprinter
