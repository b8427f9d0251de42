// HIP kernel of the batched SPRINTER decode step for gfx950: the GEMMs of 17 and more rows (prefill chunks, work lists, larger
// batches).
#include "gemm.h"
#include <algorithm>
#include <type_traits>
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
// The 256 x 256 tile is four waves of 128 x 128, one per SIMD, whose accumulators are all 256 accumulation registers: a k tile
// costs the LDS 64 KiB of fragment reads and 32 KiB of arriving loads, 768 of the 1024 cycles that its matrix instructions take at
// 128 B a cycle (eight waves of 64 x 128: 96 KiB, as many cycles as the products).  What bounds it (4096 rows): 1150 - 1180 cycles
// per k tile (eight waves: 1310 - 1410) at a clock that the power holds to 1.7 GHz in a loop of this launch and 1.9 - 2.0 in a whole
// prefill; then the epilogue, whose stores (float32) or activations no other wave hides.  In a loop of one launch, eight waves -> four, us:
// FFN-up 2 x 14336 x 4096 746 -> 722, 2 x 11008 x 4096 603 -> 563, 2 x 8192 x 2048 227 -> 229, QKV 12288 x 4096 337 -> 311,
// O-proj 4096 x 4096 113 -> 111, FFN-down 4096 x 14336 373 -> 347 (1.39 PFLOP/s).
// GELU stays on eight waves: one wave per SIMD does not hide its arithmetic (6400 x 1600 at 1811 / 2500 / 4096 rows 55.6 / 60.6 / 106.0 us;
// four waves, the epilogue through LDS as for gate + up, 60.0 / 64.7 / 114.7).
// Also measured: 32 x 32 x 16 instructions (8 - 20 % slower), a fifth stage (no faster), two fragment reads per row tile instead of
// three and a later first one (equal), 256 x 128 tiles of four waves (10 - 20 % slower but where the last round is half empty).
template <int WM, int WN, int MT, int NT, int S>
struct GemmTile {                                       // WM x WN waves, MT x NT operand tiles per wave, S stages
  static constexpr int wm = WM, wn = WN, mt = MT, nt = NT, stages = S, waves = WM * WN;
  static constexpr bool pinned = MT == 8;               // accumulators pinned to accumulation registers (256 x 256: all 256 of a wave)
};
using TileL = GemmTile<2, 2, 8, 8, 4>;                  // 256 x 256, 128 KiB: one workgroup per compute unit
using TileH = GemmTile<2, 2, 8, 4, 4>;                  // 256 x 128, for the last round of the one above
using TileG = GemmTile<4, 2, 4, 8, 4>;                  // 256 x 256 of eight waves, for GELU
using TileM = GemmTile<2, 2, 4, 4, 5>;                  // 128 x 128, 80 KiB: two
using TileS = GemmTile<2, 2, 2, 4, 6>;                  // 64 x 128, 72 KiB: two
using TileX = GemmTile<2, 2, 2, 2, 8>;                  // 64 x 64, 64 KiB: two
using TileN = GemmTile<1, 2, 2, 2, 8>;                  // 32 x 64, 48 KiB: three

// Workgroups go round-robin over the 8 XCDs: each XCD takes a contiguous run of the n_blk workgroups' work.
__device__ __forceinline__ int xcd_run(int id, int n_blk) {
  const int xcd = id & 7, q = n_blk >> 3, rem = n_blk & 7;
  return xcd * q + min(xcd, rem) + (id >> 3);
}

// Output tile (bm, bn) of share sk of SK.
template <typename T, int EPI>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, int x_tiles, int bm, int bn, int sk, int SK, void* lds) {
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr int WN = T::wn, MT = T::mt, NT = T::nt, S = T::stages;
  constexpr int TMT = T::wm * MT, TNT = WN * NT, LT = TMT + TNT, PER = LT / T::waves;   // operand tiles per stage, per wave
  constexpr int COLS = DUAL ? NT / 2 : NT;              // output column tiles of a wave (SwiGLU: gate tiles, then up tiles)
  static_assert(LT % T::waves == 0 && NT % 2 == 0 && S >= 4, "");
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  auto& ring = *reinterpret_cast<u32x4(*)[S][LT][64]>(lds);
  const int lane = threadIdx.x & 63, w = wave_index(), wm = w / WN, wn = w % WN;
  const int Kt = a.Kt;
  const void *const w_lo = a.W, *const w_up = a.W2;
  // EPI_PART: the partial product goes to part[share] (summed by the norm that follows)
  const int k0 = (int)((long long)Kt * sk / SK), k1 = (int)((long long)Kt * (sk + 1) / SK);
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
      base = up ? w_up : w_lo;
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
  int kv_b[EPI == EPI_QKV ? MT : 1], kv_slot[EPI == EPI_QKV ? MT : 1];   // the cache slots of this lane's rows
  if constexpr (EPI == EPI_QKV) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int mc = min((bm * TMT + wm * MT + i) * 16 + (lane & 15), a.rows_live - 1);
      kv_b[i] = a.kv.b[mc]; kv_slot[i] = a.kv.slot[mc];
    }
  }
#pragma unroll
  for (int i = 0; i < S - 1; ++i) issue(k0 + i);
  const int n_rows = *a.n_rows;                         // only the epilogue needs it
  Frag A, B;
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((S - 2) * PER) : "memory");
  __builtin_amdgcn_sched_barrier(0);
  read(A, k0);
  // Pinned accumulators: one wave per SIMD has nobody to hide behind, so the order of a k tile is written out - a fragment read of
  // the next k tile after every second product, a load to LDS after every NT - and the products are in asm, which keeps the
  // accumulators where they are (given the builtins in pieces, the compiler moves them between the register files: 600 moves per two
  // k tiles).  The first s_nop lies between the accumulators' initialisation and their first use.
  auto product = [&](f32x4& c, const u32x4& wf, const u32x4& xf) {
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(wf), "v"(xf));
  };
  auto step = [&](const Frag& f, Frag& nx, int kt) {
    constexpr int RPR = NT == 8 ? 3 : 2, GAP = (NT + RPR - 1) / (RPR + 1);   // fragment reads per row tile, products between them
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier\n\ts_nop 3" ::"n"((S - 3) * PER) : "memory");
    const u32x4* sn = &ring[(kt + 1 - k0) % S][0][lane];
    const size_t off = (size_t)min(kt + S - 1, k1 - 1) * 1024;
    const int slot = (kt + S - 1 - k0) % S;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        product(acc[i][j], f.w[j], f.x[i]);
        const int r = i * RPR + j / GAP;
        if (j % GAP == GAP - 1 && j / GAP < RPR && r < MT + NT) {
          if (r < NT) nx.w[r] = sn[(TMT + wn * NT + r) * 64];
          else nx.x[r - NT] = sn[(wm * MT + r - NT) * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
        if (j == NT - 1) {
#pragma unroll
          for (int q = i * PER / MT; q < (i + 1) * PER / MT; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src[q] + off),
                                             (__attribute__((address_space(3))) void*)&ring[slot][w * PER + q][0], 16, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
  };
  // The last products are on their way for some cycles more, which the compiler does not know: before anything that may read an
  // accumulator (the end of the loop is such a place).
  auto settle = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = k0;
  if constexpr (T::pinned) {
    for (; kt + 2 <= k1; kt += 2) {
      step(A, B, kt);
      step(B, A, kt + 1);
      settle();
    }
    if (kt < k1) {
      asm volatile("s_nop 3");
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) product(acc[i][j], A.w[j], A.x[i]);
      settle();
    }
  } else {
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
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // the clamped loads of the last stages still write to LDS
  // lane (lq, l16): row l16 of a row tile, columns 4 lq .. + 3 of a column tile (N is a multiple of 8)
  const int l16 = lane & 15, lq = lane >> 4;
  float* part = (EPI == EPI_PART) ? a.part + (size_t)sk * a.part_stride : nullptr;
  if constexpr (T::pinned && (EPI == EPI_F32 || EPI == EPI_PART || EPI == EPI_RESID)) {
    // float32 rows: 16 rows at a time through a wave's own piece of the ring, so that a store covers 512 bytes of a row (64 bytes of
    // 16 rows each took 10.5 us per workgroup, now 7.5)
    __syncthreads();
    constexpr int LD = NT * 16 + 4, LPR = NT * 4;       // floats per row in LDS, lanes per row
    float* buf = reinterpret_cast<float*>(&ring[0][0][0]) + w * 16 * LD;
    const int c4 = (lane % LPR) * 4, n = (bn * WN + wn) * NT * 16 + c4;
    const bool n_ok = n < a.N;
    f32x4 bias = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (EPI != EPI_PART && a.bias && n_ok) bias = *reinterpret_cast<const f32x4*>(a.bias + n);
    float* __restrict__ dst = (EPI == EPI_PART ? part : a.out_f32) + (n_ok ? n : 0);
    constexpr int RPI = 64 / LPR, NR = 16 / RPI;        // rows per instruction, instructions per row tile
    // EPI_RESID: the rows' own values, requested a row tile ahead (rows beyond the count: the last one again, dropped)
    f32x4 own[2][EPI == EPI_RESID ? NR : 1];
    auto fetch = [&](int i) {
      const int m0 = (bm * TMT + wm * MT + i) * 16;
#pragma unroll
      for (int q = 0; q < NR; ++q) own[i & 1][q] = *reinterpret_cast<const f32x4*>(dst + (size_t)max(min(m0 + q * RPI + lane / LPR, n_rows - 1), 0) * a.ldo);
    };
    if constexpr (EPI == EPI_RESID) fetch(0);
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m0 = (bm * TMT + wm * MT + i) * 16;
      if constexpr (EPI == EPI_RESID) if (i + 1 < MT) fetch(i + 1);
#pragma unroll
      for (int j = 0; j < NT; ++j) *reinterpret_cast<f32x4*>(buf + l16 * LD + j * 16 + lq * 4) = acc[i][j];
      __builtin_amdgcn_wave_barrier();                  // (LDS operations of one wave complete in order)
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const int row = q * RPI + lane / LPR, m = m0 + row;
        f32x4 v = *reinterpret_cast<const f32x4*>(buf + row * LD + c4);
        if (EPI == EPI_F32) v += bias;
        if constexpr (EPI == EPI_RESID) v = (own[i & 1][q] + bias) + v;   // the norm's order: row, bias, product
        if (m < n_rows && n_ok) *reinterpret_cast<f32x4*>(dst + (size_t)m * a.ldo) = v;
      }
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
  if constexpr (T::pinned && EPI == EPI_SWIGLU) {
    // Gate + up: two row tiles at a time into LDS, then one operand tile of the output (16 rows x 32 columns, 8 columns a lane) per
    // round of a loop that stays a loop: written out over the accumulators it is thousands of instructions, run once per workgroup and
    // fetched from L2 (the loop unrolled by 2 or 8: equal).
    __syncthreads();
    constexpr int LD = NT * 16 + 4, RT = 2, OT = COLS / 2;
    float* buf = reinterpret_cast<float*>(&ring[0][0][0]) + w * RT * 16 * LD;
#pragma unroll
    for (int i0 = 0; i0 < MT; i0 += RT) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) *reinterpret_cast<f32x4*>(buf + (i * 16 + l16) * LD + j * 16 + lq * 4) = acc[i0 + i][j];
      __builtin_amdgcn_wave_barrier();                  // (LDS operations of one wave complete in order)
#pragma unroll 1
      for (int q = 0; q < RT * OT; ++q) {
        const int i = q / OT, ct = q % OT, m = (bm * TMT + wm * MT + i0 + i) * 16 + l16, n = (bn * WN + wn) * COLS * 16 + ct * 32 + lq * 8;
        const float* p = buf + (i * 16 + l16) * LD + ct * 32 + lq * 8;
        float c[8], o[8];
        *reinterpret_cast<f32x4*>(&c[0]) = *reinterpret_cast<const f32x4*>(p);
        *reinterpret_cast<f32x4*>(&c[4]) = *reinterpret_cast<const f32x4*>(p + 4);
        const bool ok = m < n_rows && n < a.N;
        float u[8];
        *reinterpret_cast<f32x4*>(&u[0]) = *reinterpret_cast<const f32x4*>(p + COLS * 16);
        *reinterpret_cast<f32x4*>(&u[4]) = *reinterpret_cast<const f32x4*>(p + COLS * 16 + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = silu(c[e]) * u[e];
        if (ok)
          *reinterpret_cast<uint4*>((bf16_t*)a.out_act + act_idx<bf16_t>(m, n, a.out_K)) =
              make_uint4(pk_f16(o[0], o[1]), pk_f16(o[2], o[3]), pk_f16(o[4], o[5]), pk_f16(o[6], o[7]));
      }
      __builtin_amdgcn_wave_barrier();
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < COLS; ++j) {
    const int n = ((bn * WN + wn) * COLS + j) * 16 + lq * 4;
    if (n >= a.N) continue;
    float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
    if (EPI != EPI_PART && a.bias) bias = *reinterpret_cast<const float4*>(a.bias + n);
    float4 own[EPI == EPI_RESID ? MT : 1];              // (requested together; rows beyond the count: the last one again, dropped)
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
        own[i] = *reinterpret_cast<const float4*>(a.out_f32 + (size_t)max(min((bm * TMT + wm * MT + i) * 16 + l16, n_rows - 1), 0) * a.ldo + n);
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = (bm * TMT + wm * MT + i) * 16 + l16;
      if (m >= n_rows) continue;
      const f32x4 c = acc[i][j];
      if constexpr (EPI == EPI_PART) {
        *reinterpret_cast<float4*>(part + (size_t)m * a.ldo + n) = make_float4(c[0], c[1], c[2], c[3]);
      } else if constexpr (EPI == EPI_RESID) {          // the norm's order: row, bias, product
        *reinterpret_cast<float4*>(a.out_f32 + (size_t)m * a.ldo + n) = make_float4((own[i].x + bias.x) + c[0], (own[i].y + bias.y) + c[1],
                                                                                     (own[i].z + bias.z) + c[2], (own[i].w + bias.w) + c[3]);
      } else if constexpr (EPI == EPI_QKV) {
        const float o[4] = {c[0] + bias.x, c[1] + bias.y, c[2] + bias.z, c[3] + bias.w};
        if (n < a.kv.q_cols) {                          // (the three parts and a head are multiples of 4 columns)
          *reinterpret_cast<float4*>(a.out_f32 + (size_t)m * a.ldo + n) = make_float4(o[0], o[1], o[2], o[3]);
        } else {
          bf16_t* p = kv_element(a.kv, kv_b[i], kv_slot[i], n);
          if (n < a.kv.q_cols + a.kv.kv_cols) *reinterpret_cast<uint2*>(p) = make_uint2(pk_bf16(o[0], o[1]), pk_bf16(o[2], o[3]));
          else {                                        // (columns of a value tile are 8 elements apart)
#pragma unroll
            for (int e = 0; e < 4; ++e) p[8 * e] = f2bf(o[e]);
          }
        }
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

// blockIdx.y = K share (partial products).  Tiles in bands of GM row groups, so that what an XCD has in flight at a time (32 compute
// units) shares rows and columns in its own L2.
template <typename T>
__device__ __forceinline__ void tile_place(int t, int gm, int gn, int& bm, int& bn) {
  constexpr int GM = T::wm * T::mt >= 16 ? 4 : 8;
  const int band = t / (GM * gn), in_band = t - band * GM * gn, bh = min(GM, gm - band * GM);
  bm = band * GM + in_band % bh; bn = in_band / bh;
}
// whole: workgroups with a whole tile; those behind them (256 x 256 tile only) take half a tile each.
template <typename T, int EPI>
__global__ __launch_bounds__(T::waves * 64, T::pinned ? 1 : 2) void k_gemm_tile(const void* W_, const void* X_, const void* second_, int Kt_, int N_, int x_tiles, int gm, int gn, int whole,
                                                                                  const int* n_rows_, void* out_, int ldo_, int rows_live_, int half_, int shares_, size_t part_stride_,
                                                                                  GemmMore<EPI> more_) {
  GemmArgs a;                                           // second: bias, or W2; out: EPI_PART: the shares' buffer; half_: workgroups with half a tile
  a.W = W_; a.X = X_; a.W2 = second_; a.bias = EPI == EPI_SWIGLU ? nullptr : (const float*)second_; a.Kt = Kt_; a.N = N_; a.n_tiles = (N_ + 15) >> 4;
  a.n_rows = n_rows_; a.out_f32 = a.part = (float*)out_; a.out_act = out_; a.ldo = a.out_K = ldo_; a.rows_live = rows_live_; a.part_stride = part_stride_;
  if constexpr (EPI == EPI_QKV) a.kv = more_;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::stages * (T::wm * T::mt + T::wn * T::nt) * 1024];
  const int id = blockIdx.x;
  int bm, bn;
  if constexpr (T::pinned && EPI != EPI_PART) {         // (partial products: several shares, never in halves)
    if (id >= whole) {                                  // (scalar)
      const int t = xcd_run(id - whole, half_);
      tile_place<T>(whole + (t >> 1), gm, gn, bm, bn);
      gemm_tile<TileH, EPI>(a, x_tiles, bm, 2 * bn + (t & 1), 0, 1, lds);
      return;
    }
  }
  tile_place<T>(xcd_run(id, whole), gm, gn, bm, bn);
  gemm_tile<T, EPI>(a, x_tiles, bm, bn, EPI == EPI_PART ? blockIdx.y : 0, EPI == EPI_PART ? shares_ : 1, lds);
}

// Which tile, and how many K shares (partial products), for a shape: the one with the smallest estimate of
//   start + max(rounds of workgroups x cycles, padded products / rate, weights and shares / HBM rate) + the shares' way into the norm.
// Per tile: workgroups a compute unit holds, microseconds before the first product and after the last, cycles per k tile of a
// workgroup that has its compute unit for itself and what each further one adds, PFLOP/s on a full chip.  The constants are a fit to
// 1050 timings of 113 shapes (20 - 4096 rows, K 768 - 14336, N 768 - 14336, 1 - 8 shares) of the kernels before the 256 x 256 tile had four
// waves (1355 cycles and 1.22 PFLOP/s are those of eight, which GELU still takes), before a last round went out in halves and before one
// share added itself: here it counts as a partial product that the norm reads.  Against every tile and share count of the present kernels
// over 235 shapes (the products of five model pairs at 20 - 4096 rows, partial products with the norm behind them) the pick is 2.3 %
// slower than the best in the mean and 10 - 29 % at 21 of them: QKV and GELU of 4800 - 6400 columns at 140 - 300 rows (6400 x 1600 at 140
// rows 15.2 for 11.8 us), O-proj of 768 columns in two shares for one (2032 rows 19.3 for 15.7).
struct TileCost { int tm, tn, per_cu; float start_us, cycles, shared, rate; };
static float tile_us(const TileCost& c, int epi, int rows, int N, int Kt, int sk) {
  const int mats = epi == EPI_SWIGLU ? 2 : 1, cols = c.tn / mats, slots = 256 * c.per_cu;
  const int wgs = (rows + c.tm - 1) / c.tm * ((N + cols - 1) / cols) * sk, full = wgs / slots, rest = wgs % slots;
  const float kt = (float)Kt / sk, part = epi == EPI_PART ? 4.f * rows * N * sk : 0.f;
  float cycles = full * (c.cycles + c.shared * (c.per_cu - 1)) * kt;
  if (rest) cycles += (c.cycles + c.shared * ((rest + 255) / 256 - 1)) * kt;
  const float product = 2.f * wgs * c.tm * c.tn * kt * 32 / c.rate * 1e-9f, memory = (64.f * N * Kt * mats + part) / 6.3e6f;
  // the norm reads the shares at 4.5 TB/s; more than 4 take its larger variant
  return c.start_us + std::max(cycles / 2400.f, std::max(product, memory)) + part / 4.5e6f + (epi == EPI_PART && sk > 4 ? 0.3f : 0.f);
}

// One workgroup of the 256 x 256 tile runs per compute unit: a last round with work for at most half of them is dealt out in halves of
// 256 x 128, 0.6 of a round.  us: 384 tiles (6144 x 4096 at 4096 rows) 196 -> 168, 336 (3528 rows) 182 -> 152, 602 (2 x 11008 x 4096 at
// 1792 rows) 288 -> 259, 1376 (4096 rows) 596 -> 567, 1568 (2 x 14336 x 4096 at 3528 rows) 698 -> 678.
static int tiles_in_halves(int tiles) { return tiles > 256 && tiles % 256 <= 128 ? tiles % 256 : 0; }

template <typename T, int EPI>
static void launch_tile(const GemmArgs& a, int rows, int sk, hipStream_t s) {
  constexpr int tm = T::wm * T::mt * 16, cols = T::wn * T::nt * 16 / (EPI == EPI_SWIGLU ? 2 : 1);
  const int x_tiles = (int)(a.x_elems / ((size_t)a.Kt * 512)), gm = (rows + tm - 1) / tm, gn = (a.N + cols - 1) / cols;
  const int tiles = gm * gn, rest = T::pinned && sk == 1 ? tiles_in_halves(tiles) : 0, whole = tiles - rest;
  hipLaunchKernelGGL((k_gemm_tile<T, EPI>), dim3(whole + 2 * rest, sk), dim3(T::waves * 64), 0, s, a.W, a.X, EPI == EPI_SWIGLU ? a.W2 : (const void*)a.bias, a.Kt, a.N,
                     x_tiles, gm, gn, whole, a.n_rows, EPI == EPI_PART ? (void*)a.part : EPI == EPI_GELU || EPI == EPI_SWIGLU ? a.out_act : (void*)a.out_f32,
                     EPI == EPI_GELU || EPI == EPI_SWIGLU ? a.out_K : a.ldo, a.rows_live, 2 * rest, sk, a.part_stride, gemm_more<EPI>(a));
}

int gemm_tile_choice(int epi, int rows, int N, int K, int max_shares) {
  static const TileCost cost[5] = {{256, 256, 1, 8.0f, 1355.f, 0.f, 1.22f}, {128, 128, 2, 5.4f, 608.f, 465.f, 1.10f},
                                   {64, 128, 2, 4.2f, 478.f, 200.f, 0.83f}, {64, 64, 2, 3.7f, 327.f, 517.f, 0.64f},
                                   {32, 64, 3, 3.4f, 290.f, 293.f, 1.23f}};
  const int Kt = (K + 31) / 32;
  int best = 0, sk = 1;
  float best_us = 1e30f;
  for (int i = 0; i < 5; ++i)
    for (int k = 1; k <= max_shares && (k == 1 || Kt / k >= 3); ++k) {
      const float us = tile_us(cost[i], epi, rows, N, Kt, k);
      if (us < best_us) { best_us = us; best = i; sk = k; }
    }
  return best * 16 + sk;
}

template <int EPI>
static void launch_tile_epi(int tile, const GemmArgs& a, int rows, int sk, hipStream_t s) {
  switch (tile) {
    case 0: launch_tile<std::conditional_t<EPI == EPI_GELU || EPI == EPI_QKV, TileG, TileL>, EPI>(a, rows, sk, s); break;
    case 1: launch_tile<TileM, EPI>(a, rows, sk, s); break;
    case 2: launch_tile<TileS, EPI>(a, rows, sk, s); break;
    case 3: launch_tile<TileX, EPI>(a, rows, sk, s); break;
    default: launch_tile<TileN, EPI>(a, rows, sk, s); break;
  }
}

// 17 - 64 rows of an output that cannot be left in K shares: the K-split kernel of k_gemm.hip, whose 8 waves share a column tile
// (a pair of them), runs one workgroup per compute unit, so its time jumps where its 256 are exceeded - at 128 workgroups of this
// kernel's narrowest tile.  Up to there it is ahead at K from about 1000 on (8192 x 4096 at 20 / 40 / 64 rows 15.5 / 17.4 / 19.5
// against 19.3 / 19.3 / 19.5 us; 8192 x 1600 8.7 / 10.1 / 10.7 against 10.6; 2 x 4096 x 4096 14.7 / 16.4 / 19.0 against 19.5); from
// 132 on this one is, at any K (8448 x 4096 22.2 / 25.6 / 31.6 against 19.4 / 22.5 / 22.7; 8448 x 512 7.1 / 8.6 / 8.1 against 4.8 /
// 5.4 / 5.6; 2 x 4224 x 2048 12.7 / 15.0 / 17.7 against 11.3 / 12.4 / 12.5).  Partial products are ahead at any size:
// 4096 x 4096 12.2 -> 8.8 at 20 rows, 1600 x 6400 9.7 -> 6.9, 4096 x 14336 33.9 -> 24.7 at 64; and so is everything from 65 rows
// on, where that kernel takes two passes (4800 x 1600 at 80 rows 12.2 -> 9.0, 2 x 3072 x 768 9.1 -> 6.8; 12288 x 4096 36.9 / 37.4).
bool gemm_takes_tile(int epi, int N, int rows) {
  const int cols = epi == EPI_SWIGLU ? 32 : 64;
  return rows > 64 || (rows > 16 && (epi == EPI_PART || (N + cols - 1) / cols > 128));
}

// A product in one K share is added to the residual rows by its own epilogue, so that the norm that follows reads the rows alone.
// Product and norm together, us: 4096 x 4096 at 4096 rows 159 -> 148, 4096 x 14336 408 -> 389, 2048 x 2048 65.4 -> 60.4, 768 x 768 24.3 ->
// 22.8, 1500 rows of 512 x 512 11.4 -> 10.2; nowhere slower than the noise where the rule above picks one share: from 17 rows where K leaves no
// two shares of three k tiles (up to 160), from 18 - 90 at K 256 - 1600 and the widest outputs, else from a few hundred.
int launch_gemm_tile(int epi, const GemmArgs& a, int rows, int max_shares, hipStream_t s) {
  const int choice = gemm_tile_choice(epi, rows, a.N, a.K, epi == EPI_PART ? max_shares : 1), tile = choice / 16, sk = choice % 16;
  switch (epi) {
    case EPI_F32: launch_tile_epi<EPI_F32>(tile, a, rows, 1, s); return 1;
    case EPI_GELU: launch_tile_epi<EPI_GELU>(tile, a, rows, 1, s); return 1;
    case EPI_QKV: launch_tile_epi<EPI_QKV>(tile, a, rows, 1, s); return 1;
    case EPI_SWIGLU: launch_tile_epi<EPI_SWIGLU>(tile, a, rows, 1, s); return 1;
  }
  if (sk > 1) { launch_tile_epi<EPI_PART>(tile, a, rows, sk, s); return sk; }
  launch_tile_epi<EPI_RESID>(tile, a, rows, 1, s);
  return 0;
}

}  // namespace sprinter
