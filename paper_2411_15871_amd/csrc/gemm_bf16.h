// bf16 GEMM on the matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation.
//   C[M,N] (+)= opA(A) * opB(B)
// Operand layouts (all row-major):
//   TA = false: A is [M,K] (K contiguous)      TA = true: A is [K,M] (M contiguous)
//   TB = false: B is [K,N] (N contiguous)      TB = true: B is [N,K] (K contiguous)
// The forward projections use (TA=0,TB=0) with weights [in,out]; data gradients (dY * W^T) use
// (TA=0,TB=1); weight gradients (X^T * dY) use (TA=1,TB=0) and add into a float32 buffer.
//
// Two kernels: gemm_bf16_wide_kernel (256x256 tiles) takes the products that fill the chip with such tiles,
// gemm_bf16_tile_kernel (256x128 down to 64x64) the smaller ones.  This header holds the kernels and their launches, gemm_bf16.hip chooses
// among them; the sources beside it instantiate a layout each.  Common to both: a block is four waves in 2x2, one per
// SIMD, each owning a quarter of the tile; K is consumed 64 at a time from a ring of LDS stages.
//
// Operands travel global -> LDS directly (global_load_lds_dwordx4: each lane moves 16 bytes, a wave fills 1 KiB of
// consecutive LDS), so no registers or LDS-write instructions are spent on staging, and every transfer moves whole
// 128-byte lines (half lines cost a second request: the kernels before fetched rows of 64 bytes).  Because a wave's 1 KiB
// lands linearly in LDS, bank conflicts are avoided by permuting which global 16-byte chunk each lane fetches:
//   K-contiguous operand: LDS [rows][64 k], 128-byte rows; 16-byte chunk c of row r sits at c ^ ((r>>1)&7).
//   K-major operand: LDS [panels of 64 columns][64 k][64 columns]; 32-byte slot s of k-row r sits at
//   s ^ (((r>>1)&1) | ((r>>3)&1)<<1).  Its fragments come out through the transposing load ds_read_b64_tr_b16 (16 lanes
//   fetch a 4(k) x 16(column) patch, each lane receives the 4 k-values of one column; two make a fragment of 8 k).
// The transfers are inline assembly so that the compiler does not order LDS reads behind them with a full vmcnt(0) wait (it
// cannot tell stages apart); the kernels wait for them themselves, before the barrier that publishes a stage.
// Lanes whose chunk lies beyond K fetch from a 16-byte zero constant instead; rows and columns beyond the matrix are
// clamped to the last valid one (they only feed results that are never stored).
// The tile -> block mapping is XCD-aware: consecutive block ids go round-robin to the 8 XCDs, so
// block b works on logical tile (b%8)*ceil(tiles/8) + b/8, and logical tiles are ordered in groups
// of 4 tile-rows, column by column; each XCD's L2 then serves a compact 4 x n patch of tiles.
// Split-K writes float32 partial tiles to a workspace that a second kernel adds in split order, so results never depend on
// scheduling (no atomics anywhere).
// Requirements: N % 8 == 0 and every contiguous operand dimension % 8 == 0 (16-byte chunks).
#pragma once
#include <algorithm>
#include <climits>
#include <type_traits>
#include <utility>
#include "common.h"
#include "dma.h"

#define G_BK 64  // K of a stage

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

__device__ __attribute__((aligned(16))) const uint32_t dh_zero_chunk[4] = {0, 0, 0, 0};

enum { EPI_STORE_BF16 = 0, EPI_ACC_F32 = 1, EPI_PARTIAL_F32 = 2, EPI_TAIL_F32 = 3 };

struct GemmArgs {
  int M, N, K;
  const bf16_t* A;
  const bf16_t* B;
  void* C;  // bf16 (EPI_STORE_BF16), float (EPI_ACC_F32) or float partial base (EPI_PARTIAL_F32)
  int epi;
  int k_per_split;   // K handled by one split (a multiple of 64)
  int tiles_m, tiles_n, tiles_per_xcd;
  const bf16_t* bias;          // optional [N], added before the bf16 store
  const int32_t* group_rows;   // grouped GEMM: device array of row counts (blockIdx.z = group), else nullptr
  int group_mode;              // 0/1: groups split M (A and C rows), B per group; 2: groups split K, C per group
  // Modes 0/1 are issued as two launches: part 1 with the large tile, part 2 with 128x128 or 64x64 tiles.  When the groups'
  // large tiles would leave the last round of tiles over the compute units nearly empty (the row counts are data), part 1
  // keeps only each group's whole large-tile rows and part 2 takes the remainders; otherwise part 1 does everything.
  int group_part, n_groups, part1_bm, part1_bn, cus;
  // Tail launch: when the tile count leaves the last round over the compute units less than half full, those tiles
  // are issued apart with K split over blockIdx.y, so that the round is short; tile_first = launch index of this
  // launch's first tile; EPI_TAIL_F32 writes tile-local float32 partials [split][tile][BM][BN].
  int tile_first;
  // SwiGLU fused into the epilogue (bf16 result).  GLU_FWD: the GEMM is the gate/up projection with N = 2*glu_f columns
  // [gate | up], glu_f % 128 == 0; half of a tile's columns are gate columns, the other half the up columns of the same outputs
  // (its B panel is fetched from two places); it stores both to C and gate*sigmoid(gate)*up to glu_out [M, glu_f].  GLU_BWD: the GEMM yields dA [M, N = glu_f]; instead of storing it the epilogue reads gate/up from glu_in
  // [M, 2*glu_f] and stores d(gate), d(up) to C [M, 2*glu_f].  Element arithmetic: swiglu_*_elem, as the row-wise kernels.
  int glu_mode, glu_f;
  const bf16_t* glu_in;
  bf16_t* glu_out;
  // An all-reduce stand-in carried along (Sec. 6.3, Table 7's closing remark: computation and communication in one kernel,
  // their shares of the machine fixed inside it instead of left to the dispatcher): the first ar_blocks thread blocks of
  // the launch stream the payload -- they hold their compute units for as long as the transfer lasts --, the tiles
  // follow.  0 = none.
  int ar_blocks;
  int n_split;  // > 1: K splits of a launch whose index range covers splits x tiles, split after split (0: split = blockIdx.y)
  int k_chain;  // K range a block sums on its own before it joins the total (a multiple of G_BK, see g_check_chain; 0: the whole split)
};
// The stand-in's operands travel as a kernel argument of their own: GemmArgs is edited by the grouped path and lives in
// registers, the partial pointers are indexed at run time and stay in the argument segment.
struct GemmAr {
  int ranks;
  size_t n8;
  bf16_t* out;
  PartPtrs parts;
};
enum { GLU_NONE = 0, GLU_FWD = 1, GLU_BWD = 2 };

// Launch index -> tile coordinates.  XCD-aware: launch indices go round-robin over the 8 XCDs, each XCD owns a
// contiguous range of the logical tile order, which walks the tiles in bands of 4 tile rows.
__device__ __forceinline__ bool tile_of_logical(int logical, int tiles_m, int tiles_n, int& tm, int& tn) {
  if (logical >= tiles_m * tiles_n) return false;
  const int group = logical / (4 * tiles_n);
  const int rows_in_group = min(4, tiles_m - group * 4);
  const int in_group = logical - group * 4 * tiles_n;
  tm = group * 4 + in_group % rows_in_group;
  tn = in_group / rows_in_group;
  return true;
}
__device__ __forceinline__ bool tile_of_launch(int idx, int tiles_m, int tiles_n, int tiles_per_xcd, int& tm, int& tn) {
  if ((idx >> 3) >= tiles_per_xcd) return false;  // grouped launches: grid sized for the largest group
  return tile_of_logical((idx & 7) * tiles_per_xcd + (idx >> 3), tiles_m, tiles_n, tm, tn);
}
// Whether the remainders go to part 2: decided from the device-side row counts, the same way by both launches.
__device__ __forceinline__ bool grouped_split_remainders(const GemmArgs& g) {
  int full = 0, bulk = 0;
  const int tn = (g.N + g.part1_bn - 1) / g.part1_bn;
  for (int i = 0; i < g.n_groups; i++) {
    const int r = g.group_rows[i];
    full += (r + g.part1_bm - 1) / g.part1_bm * tn;
    bulk += r / g.part1_bm * tn;
  }
  const int tail = full % g.cus;  // tiles of the last, partly filled round
  return tail != 0 && tail * 4 < g.cus && bulk <= full / g.cus * g.cus;
}

// Grouped launches: the groups' rows lie behind one another; this block's group is blockIdx.z.  The row counts are data
// (expert routing), so the extents are fixed up here from device memory and the grid is sized for the largest possible
// group; surplus blocks leave at the tile check.  False: this block has nothing to do.
template <int BM>
__device__ __forceinline__ bool group_setup(GemmArgs& g) {
  int row0 = 0;
  for (int i = 0; i < (int)blockIdx.z; i++) row0 += g.group_rows[i];
  int rows = g.group_rows[blockIdx.z];
  if (g.group_part != 0) {
    const bool split = grouped_split_remainders(g);
    if (g.group_part == 1) {
      if (split) rows -= rows % g.part1_bm;
    } else {
      if (!split) return false;
      row0 += rows - rows % g.part1_bm;
      rows %= g.part1_bm;
    }
  }
  row0 = __builtin_amdgcn_readfirstlane(row0);  // the same in every lane, as the compiler may not know of loaded values
  rows = __builtin_amdgcn_readfirstlane(rows);
  if (rows == 0) return false;
  if (g.group_mode == 2) {
    g.A += (size_t)row0 * g.M;
    g.B += (size_t)row0 * g.N;
    g.C = reinterpret_cast<float*>(g.C) + (size_t)blockIdx.z * g.M * g.N;
    g.K = rows;
    g.k_per_split = rows;
  } else {
    g.A += (size_t)row0 * g.K;
    g.B += (size_t)blockIdx.z * g.K * g.N;
    g.C = reinterpret_cast<bf16_t*>(g.C) + (size_t)row0 * g.N;
    g.M = rows;
    g.tiles_m = (rows + BM - 1) / BM;
    g.tiles_per_xcd = (g.tiles_m * g.tiles_n + 7) / 8;
  }
  return true;
}

// ------------------------------------------------------------------------------------ operand tiles in LDS
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
#define G_PIN() __builtin_amdgcn_sched_barrier(0)

// Transfers a wave makes for its share of a stage, and the operand's bytes of the stage.  A K-major tile of 32 columns more than
// whole panels (ROWS = 96, 160, 224) takes a whole panel's room for them: the lanes of the missing half fetch the columns that are
// there once more (the same lines), so that every panel has one layout.
template <int ROWS, bool KMAJOR> constexpr int g_transfers = KMAJOR ? (ROWS + 63) / 64 * 2 : ROWS / 32;
template <int ROWS, bool KMAJOR> constexpr int g_bytes = g_transfers<ROWS, KMAJOR> * 4096;
template <int ROWS, bool KMAJOR> using GOffsets = uint32_t[g_transfers<ROWS, KMAJOR>];
// Row of the operand's non-K dimension (relative to the tile of ROWS) and k of the 16-byte chunk lane `lane` fetches in
// transfer j of wave `wave`.
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ void g_chunk(int wave, int j, int lane, int& r, int& k) {
  const int inst = wave * g_transfers<ROWS, KMAJOR> + j;
  if (KMAJOR) {
    k = (inst & 7) * 8 + (lane >> 3);
    const int slot = ((lane & 7) >> 1) ^ (((k >> 1) & 1) | (((k >> 3) & 1) << 1));
    r = (inst >> 3) * 64 + slot * 16 + (lane & 1) * 8;
    if (ROWS % 64 != 0 && r >= ROWS) r -= 32;
  } else {
    r = inst * 8 + (lane >> 3);
    k = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
  }
}
// Byte offsets relative to the tile's origin.  half_jump: the tile's second half of columns lies that many columns further on.
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ void g_offsets(GOffsets<ROWS, KMAJOR>& voff, int r0, int R, int K, int wave, int lane, int half_jump = 0) {
#pragma unroll
  for (int j = 0; j < g_transfers<ROWS, KMAJOR>; j++) {
    int r, k;
    g_chunk<ROWS, KMAJOR>(wave, j, lane, r, k);
    if (KMAJOR) {
      const int col = half_jump != 0 ? r + (r >= ROWS / 2 ? half_jump : 0) : min(r0 + r, R - 8) - r0;
      voff[j] = (uint32_t)(((size_t)k * R + col) * sizeof(bf16_t));
    } else {
      voff[j] = (uint32_t)(((size_t)(min(r0 + r, R - 1) - r0) * K + k) * sizeof(bf16_t));
    }
  }
}
// A stage that reaches beyond k_end: chunks there come from the zero constant.  K: the operand's row pitch if K-contiguous.
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ void g_issue_ragged(uint32_t lds_wave, const bf16_t* __restrict__ base, int r0, int k0, int R, int K, int k_end,
                                               int wave, int lane, int half_jump = 0) {
  asm volatile("" : "+v"(lane));  // computed here: shared with the steady path's offsets it would hold registers through the main loop
#pragma unroll
  for (int j = 0; j < g_transfers<ROWS, KMAJOR>; j++) {
    int r, k;
    g_chunk<ROWS, KMAJOR>(wave, j, lane, r, k);
    r += r0 + (r >= ROWS / 2 ? half_jump : 0);
    k += k0;
    const bf16_t* src = (r < R && k < k_end) ? base + (KMAJOR ? (size_t)k * R + r : (size_t)r * K + k) : reinterpret_cast<const bf16_t*>(dh_zero_chunk);
    dma16(src, lds_wave + j * 1024);
  }
}
// A stage's transfers from offsets made by g_offsets: transfer j carries the constant j KiB - G_BIAS, which the hardware adds to its
// memory and to its LDS address (see dma.h).  So the LDS address is set once per operand and a transfer is one instruction instead
// of four, which a lone wave's products left no room for (128x128, stage of 32 products: 128 -> 103 instructions).
#define G_BIAS 4096
template <int N>
__device__ __forceinline__ void g_bias_transfers(const char*& base, uint32_t (&voff)[N]) {
  base -= G_BIAS;
#pragma unroll
  for (int j = 0; j < N; j++) voff[j] += 2 * G_BIAS - j * 1024;
}
template <int N>
__device__ __forceinline__ void g_transfers_of_stage(uint32_t lds, const char* base, const uint32_t (&voff)[N]) {
  const uint32_t m = dma_lds(lds + G_BIAS);
#pragma unroll
  for (int j = 0; j < N; j++) dma16_at(m, base, voff[j], j * 1024 - G_BIAS);
}
// Lane pointers of a wave whose first 16-row tile is tile0: K-contiguous one per k-step of 32, K-major one per tile modulo 4.
template <bool KMAJOR>
__device__ __forceinline__ void g_pointers(const lds_char* (&p)[4], const lds_char* base, int tile0, int lane) {
  const int l16 = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int x = 0; x < 4; x++) {
    if (KMAJOR) {  // lane l16 of a group fetches k-row kg*8 + l16/4 (and the one 4 further), 4 columns
      const int kr = kg * 8 + (l16 >> 2), t = tile0 + x;
      p[x] = base + (t >> 2) * 8192 + kr * 128 + ((t & 3) ^ (((kr >> 1) & 1) | (((kr >> 3) & 1) << 1))) * 32 + (l16 & 3) * 8;
    } else {       // row l16, chunk ks*4 + kg
      p[x] = base + (tile0 * 16 + l16) * 128 + ((((x & 1) * 4 + kg) ^ ((l16 >> 1) & 7)) << 4);
    }
  }
}
// Fragment of 16 rows (tile i of the wave) and 32 k (step ks of the stage), `stage` bytes behind the pointers.
template <bool KMAJOR>
__device__ __forceinline__ bf16x8 g_frag(const lds_char* const (&p)[4], int ks, int i, int stage = 0) {
  if (!KMAJOR) return *reinterpret_cast<const lds_bf16x8*>(p[ks] + stage + i * 2048);
  const lds_char* q = p[i & 3] + stage + (i >> 2) * 8192 + ks * 4096;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)q);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + 512));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}
// A wave-uniform pointer, told to the compiler so that it stays in scalar registers.
__device__ __forceinline__ const char* g_uniform(const char* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}

// acc += A * B with the accumulator tied to one AGPR quad: the 256x256 kernel's accumulators fill that half of the register
// file exactly, and through the intrinsic (whose result may land elsewhere) the compiler moves them around inside the
// loop.  The operands come straight from LDS reads, so no vector-ALU write precedes the instruction closely; g_settle()
// covers the result's latency before anything else reads an accumulator.
__device__ __forceinline__ void g_mfma(f32x4& acc, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
template <int MT, int NT>
__device__ __forceinline__ void g_settle(f32x4 (&acc)[MT][NT]) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < MT; i++)
#pragma unroll
    for (int j = 0; j < NT; j++) asm volatile("" : "+a"(acc[i][j]));
}

// Epilogue of a block of 2x2 waves, each holding MT x NT tiles of 16x16: acc[i][j][e] = C[row i*16 + lane%16][column j*16 +
// 4*(lane/16) + e] of the wave's part (the operands go in swapped, so a lane holds 4 consecutive columns of one row).  It is
// turned around in LDS (wave-private regions; the stages are free) so that a lane stores 16 bytes of a contiguous row segment.
template <int MT, int NT, bool F32OUT>
__device__ __forceinline__ void g_epilogue(const GemmArgs& g, f32x4 (&acc)[MT][NT], unsigned char* smem_raw, int wave, int lane, int m0, int n0, int split,
                                           bool glu_fwd, int nb0) {
  constexpr int WM = MT * 16, WN = NT * 16, BM = 2 * WM, BN = 2 * WN;
  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN, l16 = lane & 15, kg = lane >> 4;
  g_settle(acc);
  __syncthreads();
  if constexpr (F32OUT) {
    constexpr int PASSES = WM / 8, U = PASSES % 8 == 0 ? 8 : PASSES % 6 == 0 ? 6 : PASSES, UNITS = PASSES / U;  // 8 rows a pass, U passes a unit
    const int r8 = lane >> 3, ch = lane & 7;
    float* Cf = reinterpret_cast<float*>(g.C);
    size_t ld = g.N;
    int row0 = m0 + wm0, col0 = n0 + wn0, rows = g.M, cols = g.N;
    if (g.epi == EPI_PARTIAL_F32) Cf += (size_t)split * g.M * g.N;
    if (g.epi == EPI_TAIL_F32) {  // whole tile, tile-local layout (rows/columns beyond the matrix are never read back)
      Cf += ((size_t)split * gridDim.x + blockIdx.x) * (BM * BN);
      ld = BN; row0 = wm0; col0 = wn0; rows = BM; cols = BN;
    }
    const bool add = g.epi == EPI_ACC_F32;
    float* reg = reinterpret_cast<float*>(smem_raw) + wave * (WM * 32);  // [WM rows][32 columns], chunks swizzled by row
    f32x4 old[2][U];  // C of a unit, fetched one unit ahead
    auto at = [&](int j, int it) { return Cf + (size_t)(row0 + it * 8 + r8) * ld + col0 + j * 32 + ch * 4; };
    auto in = [&](int j, int it) { return row0 + it * 8 + r8 < rows && col0 + j * 32 + ch * 4 < cols; };
    auto fetch = [&](int x) {
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int j = x / UNITS, it = (x % UNITS) * U + u;
        old[x & 1][u] = add && in(j, it) ? *reinterpret_cast<const f32x4*>(at(j, it)) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    };
    fetch(0);
#pragma unroll
    for (int x = 0; x < UNITS * (WN / 32); x++) {
      const int j = x / UNITS;
      if (x + 1 < UNITS * (WN / 32)) fetch(x + 1);
      if (x % UNITS == 0) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < MT; i++) {
#pragma unroll
          for (int q = 0; q < 2; q++) {
            const int row = i * 16 + l16, c = 4 * q + kg;
            *reinterpret_cast<f32x4*>(reg + row * 32 + ((c ^ (row & 7)) << 2)) = acc[i][j * 2 + q];
          }
          G_PIN();
        }
        __builtin_amdgcn_wave_barrier();
      }
#pragma unroll
      for (int u = 0; u < U; u++) {
        const int it = (x % UNITS) * U + u, row = it * 8 + r8;
        const f32x4 v = *reinterpret_cast<const f32x4*>(reg + row * 32 + ((ch ^ (row & 7)) << 2));
        if (in(j, it)) *reinterpret_cast<f32x4*>(at(j, it)) = add ? old[x & 1][u] + v : v;
      }
      G_PIN();
    }
  } else {
    constexpr int SW = WN < 64 ? WN : 64, CPR = SW / 8, RPP = 64 / CPR;  // slab of columns, its 16-byte chunks per row, rows a pass
    const int rr = lane / CPR, ch = lane % CPR;
    bf16_t* Cb = reinterpret_cast<bf16_t*>(g.C);
    bf16_t* reg = reinterpret_cast<bf16_t*>(smem_raw) + wave * (WM * WN);  // slabs of [WM rows][SW columns]
#pragma unroll
    for (int hh = 0; hh < WN / SW; hh++) {
      bf16_t* rh = reg + hh * (WM * SW);
#pragma unroll
      for (int j = 0; j < SW / 16; j++) {
        const int c0 = j * 16 + 4 * kg;
        f32x4 bias = {0.f, 0.f, 0.f, 0.f};
        if (g.bias != nullptr && n0 + wn0 + hh * SW + c0 < g.N) {
          const bf16x4 bb = *reinterpret_cast<const bf16x4*>(g.bias + n0 + wn0 + hh * SW + c0);
          bias = f32x4{(float)bb[0], (float)bb[1], (float)bb[2], (float)bb[3]};
        }
#pragma unroll
        for (int i = 0; i < MT; i++) {
          const int row = i * 16 + l16;
          const f32x4 v = acc[i][hh * (SW / 16) + j] + bias;
          const bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
          *reinterpret_cast<bf16x4*>(rh + row * SW + ((((c0 >> 3) ^ (row & (CPR - 1))) << 3) | (c0 & 4))) = o;
        }
        G_PIN();
      }
      __builtin_amdgcn_wave_barrier();
      if (g.glu_mode != GLU_BWD) {
        // gate/up projection: wave column 0 holds gate columns, wave column 1 the up columns of outputs nb0 + ...
        const int cb = (glu_fwd ? nb0 + (wave & 1) * g.glu_f : n0 + wn0) + hh * SW + ch * 8;
#pragma unroll
        for (int it = 0; it < WM / RPP; it++) {
          const int row = it * RPP + rr;
          const bf16x8 o = *reinterpret_cast<const bf16x8*>(rh + row * SW + ((ch ^ (row & (CPR - 1))) << 3));
          if (m0 + wm0 + row < g.M && cb < g.N) *reinterpret_cast<bf16x8*>(Cb + (size_t)(m0 + wm0 + row) * g.N + cb) = o;
          if ((it & 3) == 3) G_PIN();
        }
      }
    }
    if (glu_fwd) {
      // once both waves of a row have written, each combines half of the rows (the values as stored, i.e. rounded to bf16)
      __syncthreads();
      const bf16_t* rg = reinterpret_cast<const bf16_t*>(smem_raw) + (wave & 2) * (WM * WN);
      const bf16_t* ru = rg + WM * WN;
#pragma unroll 1
      for (int hh = 0; hh < WN / SW; hh++)
#pragma unroll 2
        for (int it = 0; it < WM / RPP / 2; it++) {
          const int row = (wave & 1) * (WM / 2) + it * RPP + rr, off = hh * (WM * SW) + row * SW + ((ch ^ (row & (CPR - 1))) << 3);
          const bf16x8 gv = *reinterpret_cast<const bf16x8*>(rg + off), uv = *reinterpret_cast<const bf16x8*>(ru + off);
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 8; e++) o[e] = (bf16_t)swiglu_fwd_elem((float)gv[e], (float)uv[e]);
          if (m0 + wm0 + row < g.M) *reinterpret_cast<bf16x8*>(g.glu_out + (size_t)(m0 + wm0 + row) * g.glu_f + nb0 + hh * SW + ch * 8) = o;
          G_PIN();
        }
    }
    if (g.glu_mode == GLU_BWD) {
      // gate/up of several passes are fetched together, so that the epilogue waits for memory once per batch
      constexpr int PASSES = WM / RPP, NB = PASSES % 8 == 0 ? 8 : PASSES % 6 == 0 ? 6 : PASSES;
#pragma unroll 1
      for (int hh = 0; hh < WN / SW; hh++)
#pragma unroll 1
        for (int it0 = 0; it0 < PASSES; it0 += NB) {
          bf16x8 gv[NB], uv[NB];
#pragma unroll
          for (int u = 0; u < NB; u++) {
            const size_t r2 = (size_t)min(m0 + wm0 + (it0 + u) * RPP + rr, g.M - 1) * (2 * (size_t)g.glu_f) + min(n0 + wn0 + hh * SW + ch * 8, g.glu_f - 8);
            gv[u] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(g.glu_in + r2));
            uv[u] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(g.glu_in + r2 + g.glu_f));
          }
#pragma unroll
          for (int u = 0; u < NB; u++) {
            const int row = (it0 + u) * RPP + rr;
            const int cb = n0 + wn0 + hh * SW + ch * 8;
            const size_t r2 = (size_t)(m0 + wm0 + row) * (2 * (size_t)g.glu_f) + cb;
            const bf16x8 o = *reinterpret_cast<const bf16x8*>(reg + hh * (WM * SW) + row * SW + ((ch ^ (row & (CPR - 1))) << 3));
            bf16x8 dg, du;
#pragma unroll
            for (int e = 0; e < 8; e++) {
              float a, b;
              swiglu_bwd_elem((float)gv[u][e], (float)uv[u][e], (float)o[e], a, b);
              dg[e] = (bf16_t)a;
              du[e] = (bf16_t)b;
            }
            if (m0 + wm0 + row < g.M && cb < g.glu_f) {
              *reinterpret_cast<bf16x8*>(Cb + r2) = dg;
              *reinterpret_cast<bf16x8*>(Cb + r2 + g.glu_f) = du;
            }
            G_PIN();
          }
        }
    }
  }
}

// The first blocks of a launch that carries a stand-in are shares of the stand-in, not tiles: true in these once they are through.
__device__ __forceinline__ bool g_standin_block(const GemmArgs& g, const GemmAr& ar) {
  if (g.ar_blocks == 0 || blockIdx.x >= (unsigned)g.ar_blocks) return false;
  if (blockIdx.y == 0 && blockIdx.z == 0)
    allreduce_span<bf16_t>(ar.parts, ar.ranks, ar.out, ar.n8, (size_t)blockIdx.x * blockDim.x + threadIdx.x, (size_t)g.ar_blocks * blockDim.x);
  return true;
}
// What block bx of a product's tiles works on: false if it has no tile (it is surplus).
struct GemmTile {
  int m0, n0, tn, split, k_begin, n, n_full, k_end;  // n: stages of its K range, of which the first n_full are whole
};
template <int BM, int BN>
__device__ __forceinline__ bool g_begin(GemmArgs& g, int bx, GemmTile& w) {
  if (g.group_rows != nullptr && !group_setup<BM>(g)) return false;
  int tm;
  w.split = blockIdx.y;
  if (g.n_split > 1) {  // contiguous ranges again: an XCD works on neighbouring tiles of the same K range
    const int n = g.tiles_m * g.tiles_n, logical = (bx & 7) * g.tiles_per_xcd + (bx >> 3);
    w.split = __builtin_amdgcn_readfirstlane(logical / n);
    if (w.split >= g.n_split) return false;
    tile_of_logical(logical - w.split * n, g.tiles_m, g.tiles_n, tm, w.tn);
  } else if (!tile_of_launch(bx + g.tile_first, g.tiles_m, g.tiles_n, g.tiles_per_xcd, tm, w.tn)) {
    return false;
  }
  w.m0 = tm * BM;
  w.n0 = w.tn * BN;
  w.k_begin = w.split * g.k_per_split;
  w.k_end = min(g.K, w.k_begin + g.k_per_split);
  w.n = max(0, (w.k_end - w.k_begin + G_BK - 1) / G_BK);
  w.n_full = max(0, (w.k_end - w.k_begin) / G_BK);
  return true;
}
#define G_VMCNT(n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory")

// ------------------------------------------------------------------------------------ 256x256 tiles
// Bound: the matrix cores under the chip's power limit.  At 8192^3 they are 81 % busy (A transposed with float32 accumulation:
// 71 %) at the clock that power allows, 1.4 to 1.9 GHz, so
// energy per product counts as much as idle cycles: the 16x16x32 instruction (half the accumulator traffic of
// 32x32x16 per product), 128x128 wave tiles (a third fewer LDS reads than 128x64) and whole-line transfers
// each raised the clock at the same utilisation.  Measured against an 8-wave kernel with 128x64 wave tiles, 32x32x16
// instructions and K tiles of 32 (same box, N(0,1) operands, a steady sequence; the first tens of launches after idling take
// 10-15 % longer, operands of zeros 12 % less): 8192^3 832 -> 723 us (1520 TFLOP/s), B transposed 880 -> 727, A transposed
// with float32 accumulation 889 -> 785; 4096x3584x4096 100 -> 86 us; 4096x4096x1792 53 -> 46 us.  With 32x32x16
// instructions in the same schedule: 766 us at 8192^3.
// The large-tile kernel: four waves, one per SIMD, each owning a 128x128 part of C (256 accumulator registers in AGPRs).
// K is consumed 64 at a time.  A K tile is worked off in four quadrants (a0 b0, a0 b1, a1 b1, a1 b0: halves of 64 rows / columns of a wave's
// part); the fragments of the half that comes next are read while the current quadrant's products are issued.  So the first halves of A and B are read
// in the third and fourth quadrant of the tile before and the second halves in the first two, and the LDS is a ring of four slots of 32 KiB, each the same half of both
// operands: after each second quadrant a barrier publishes the next slot and frees the one just read, whose refill follows.  A transfer has one and a half
// tiles (about 2 us) until it is needed; as a ring of two whole tiles it had half a tile to one, less than the memory's latency while another
// strand's kernels load it, and in launches of several rounds, whose blocks run out of step and miss the L2 more often.  Measured against that ring (us): Llama-70B
// shard's gate/up products 712 -> 669 (forward), 659 -> 622 (data gradient), 780 -> 733 (weight gradient), its interleaved step 6100 -> 5797; 8192^3 alone 1530
// TFLOP/s either way.  A fifth slot (all of the LDS): the step 1 % slower.  Matrix instructions, LDS reads and transfers are
// interleaved two products at a time and pinned in that order.
#define GW_SLOT 32768u
#define GW_RING 4

// Half h of a 256-wide operand tile: the 64 rows (columns) h*64 .. h*64+63 of either wave row (wave column).  Tile index of the half's u-th.
__device__ __forceinline__ int gw_row(int h, int u) { return (u >> 6) * 128 + h * 64 + (u & 63); }
// Offsets of a wave's transfers of both halves, four each; as g_offsets.
template <bool KMAJOR>
__device__ __forceinline__ void gw_offsets(uint32_t (&voff)[8], int r0, int R, int K, int wave, int lane, int half_jump = 0) {
#pragma unroll
  for (int x = 0; x < 8; x++) {
    int u, k;
    g_chunk<128, KMAJOR>(wave, x & 3, lane, u, k);
    const int r = gw_row(x >> 2, u);
    if (KMAJOR) {
      const int col = half_jump != 0 ? r + (r >= 128 ? half_jump : 0) : min(r0 + r, R - 8) - r0;
      voff[x] = (uint32_t)(((size_t)k * R + col) * sizeof(bf16_t));
    } else {
      voff[x] = (uint32_t)(((size_t)(min(r0 + r, R - 1) - r0) * K + k) * sizeof(bf16_t));
    }
    voff[x] += 2 * G_BIAS - (x & 3) * 1024;  // see g_bias_transfers
  }
}
// Half h of a stage that reaches beyond k_end; as g_issue_ragged.
template <bool KMAJOR>
__device__ __forceinline__ void gw_issue_ragged(uint32_t lds_wave, const bf16_t* __restrict__ base, int h, int r0, int k0, int R, int K, int k_end, int wave,
                                                int lane, int half_jump = 0) {
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int j = 0; j < 4; j++) {
    int u, k;
    g_chunk<128, KMAJOR>(wave, j, lane, u, k);
    int r = gw_row(h, u);
    r += r0 + (r >= 128 ? half_jump : 0);
    k += k0;
    const bf16_t* src = (r < R && k < k_end) ? base + (KMAJOR ? (size_t)k * R + r : (size_t)r * K + k) : reinterpret_cast<const bf16_t*>(dh_zero_chunk);
    dma16(src, lds_wave + j * 1024);
  }
}

template <bool TA, bool TB, bool F32OUT>
__global__ __launch_bounds__(256, 1) void gemm_bf16_wide_kernel(GemmArgs g, const GemmAr ar) {
  // Weight gradients claim 500 registers: with the 484 they need, blocks of up to 24 registers fit beside them (a Send/Recv stand-in's 8), and the launch waits
  // for the tiles that share their unit: 224 tiles beside such an exchange 119 us, sharing 136; the context-parallel 8B step 1360 and 1376.
  if (TA) asm volatile("" ::: "v240");
  if (g_standin_block(g, ar)) return;
  GemmTile w;
  if (!g_begin<256, 256>(g, (int)blockIdx.x - g.ar_blocks, w)) return;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool glu_fwd = !TA && !TB && !F32OUT && g.glu_mode == GLU_FWD;
  const int jump = glu_fwd ? g.glu_f - 128 : 0;  // B panel: 128 gate columns, then the 128 up columns of the same outputs
  const int nb0 = glu_fwd ? w.tn * 128 : w.n0, n = w.n, n_full = w.n_full;

  uint32_t voa[8], vob[8];
  gw_offsets<TA>(voa, w.m0, g.M, g.K, wave, lane);
  gw_offsets<!TB>(vob, nb0, g.N, g.K, wave, lane, jump);
  const size_t sa = (TA ? (size_t)G_BK * g.M : (size_t)G_BK) * sizeof(bf16_t);
  const size_t sb = (TB ? (size_t)G_BK : (size_t)G_BK * g.N) * sizeof(bf16_t);
  // next tile to transfer
  const char* ap = g_uniform(reinterpret_cast<const char*>(g.A + (TA ? (size_t)w.k_begin * g.M + w.m0 : (size_t)w.m0 * g.K + w.k_begin))) - G_BIAS;
  const char* bp = g_uniform(reinterpret_cast<const char*>(g.B + (TB ? (size_t)nb0 * g.K + w.k_begin : (size_t)w.k_begin * g.N + nb0))) - G_BIAS;
  const uint32_t lds0 = lds_address(smem_raw) + wave * 4096u;
  // Half h of tile t: A's half in the first 16 KiB of its slot, B's in the second.
  auto issue = [&](int t, int h) {
    const uint32_t slot = lds0 + ((t & 1) * 2 + h) * GW_SLOT;
    if (t < n_full) {
      const uint32_t ma = dma_lds(slot + G_BIAS);
#pragma unroll
      for (int j = 0; j < 4; j++) dma16_at(ma, ap, voa[h * 4 + j], j * 1024 - G_BIAS);
      const uint32_t mb = dma_lds(slot + 16384u + G_BIAS);
#pragma unroll
      for (int j = 0; j < 4; j++) dma16_at(mb, bp, vob[h * 4 + j], j * 1024 - G_BIAS);
    } else {
      gw_issue_ragged<TA>(slot, g.A, h, w.m0, w.k_begin + t * G_BK, g.M, g.K, w.k_end, wave, lane);
      gw_issue_ragged<!TB>(slot + 16384u, g.B, h, nb0, w.k_begin + t * G_BK, g.N, g.K, w.k_end, wave, lane, jump);
    }
  };
  if (n > 0) { issue(0, 0); issue(0, 1); }
  ap += sa;
  bp += sb;
  if (n > 1) { issue(1, 0); issue(1, 1); }
  ap += sa;
  bp += sb;

  f32x4 acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int j = 0; j < 8; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  g_settle(acc);
  const lds_char* pa[4];
  const lds_char* pb[4];
  g_pointers<TA>(pa, (const lds_char*)smem_raw, (wave >> 1) * 4, lane);
  g_pointers<!TB>(pb, (const lds_char*)smem_raw + 16384, (wave & 1) * 4, lane);

  bf16x8 fa0[8], fa1[8], fbx[8], fby[8];  // halves of 64 rows / columns: [k-step of 32][16-row tile]
  auto rd_a = [&](int half, int e) { return g_frag<TA>(pa, e >> 2, e & 3, half * (int)GW_SLOT); };
  auto rd_b = [&](int half, int e) { return g_frag<!TB>(pb, e >> 2, e & 3, half * (int)GW_SLOT); };
  auto shift = [&](const lds_char* (&p)[4], int d) {
#pragma unroll
    for (int x = 0; x < 4; x++) p[x] += d;
  };
  // operands swapped: the result tile is C^T, so a lane holds 4 consecutive columns of one row
  auto quad = [&](const bf16x8 (&a)[8], const bf16x8 (&b)[8], int ah, int bh, auto aux) {
#pragma unroll
    for (int i = 0; i < 16; i++) {
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const int m = i * 2 + u, ks = m >> 4, x = (m >> 2) & 3, y = m & 3;
        g_mfma(acc[ah * 4 + x][bh * 4 + y], b[ks * 4 + y], a[ks * 4 + x]);
      }
      aux(i);
      G_PIN();
    }
  };
  // Everything up to this half has landed and every wave is through with the half before it: at most LATER transfers, those of
  // halves further on, are still under way.
#define GW_PUBLISH(LATER) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LATER) : "memory")
  if (n > 0) {
    if (n > 1) G_VMCNT(24); else G_VMCNT(8);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; e++) { fa0[e] = rd_a(0, e); fbx[e] = rd_b(0, e); }
    if (n > 1) GW_PUBLISH(16); else GW_PUBLISH(0);
  }
  int t = 0;
  // Works off tile t, of parity S.  f0 holds the fragments of its first B half, f1 receives those of the second and then
  // the next tile's first half.  STEADY: tile t+2 is a full tile, its transfers go out between the products.
  auto step = [&](auto stage, auto steady, bf16x8 (&f0)[8], bf16x8 (&f1)[8]) {
    constexpr int S = decltype(stage)::value;
    constexpr bool STEADY = decltype(steady)::value;
    constexpr int to_next = S == 0 ? (int)(2 * GW_SLOT) : -(int)(2 * GW_SLOT);
    const bool later = t + 2 < n;
    uint32_t m = 0;
    auto transfer = [&](int i, int h) {  // the i-th transfer of half h of tile t+2
      if (i == 0) m = dma_lds(lds0 + (S * 2 + h) * GW_SLOT + G_BIAS);
      if (i == 4) m = dma_lds(lds0 + (S * 2 + h) * GW_SLOT + 16384u + G_BIAS);
      if (i < 4) dma16_at(m, ap, voa[h * 4 + i], i * 1024 - G_BIAS);
      else dma16_at(m, bp, vob[h * 4 + i - 4], (i - 4) * 1024 - G_BIAS);
    };
    if (!STEADY && later) issue(t + 2, 0);
    quad(fa0, f0, 0, 0, [&](int i) {
      if ((i & 1) == 0) f1[i >> 1] = rd_b(1, i >> 1);
      else if (STEADY) transfer(i >> 1, 0);
    });
    quad(fa0, f1, 0, 1, [&](int i) {
      if (i < 8) fa1[i] = rd_a(1, i);
      if (i == 13) {
        if (STEADY || later) GW_PUBLISH(16); else GW_PUBLISH(8);
      }
    });
    shift(pa, to_next);
    shift(pb, to_next);
    if (!STEADY && later) issue(t + 2, 1);
    quad(fa1, f1, 1, 1, [&](int i) {
      if ((i & 1) == 0) fa0[i >> 1] = rd_a(0, i >> 1);
      else if (STEADY) transfer(i >> 1, 1);
    });
    quad(fa1, f0, 1, 0, [&](int i) {
      if (i < 8) f1[i] = rd_b(0, i);
      if (i == 13) {
        if (STEADY || later) GW_PUBLISH(16); else GW_PUBLISH(0);
      }
    });
    ap += sa;
    bp += sb;
  };
  const std::integral_constant<int, 0> s0{};
  const std::integral_constant<int, 1> s1{};
  for (; t + 4 <= n_full; t += 2) {
    step(s0, std::true_type{}, fbx, fby);
    step(s1, std::true_type{}, fby, fbx);
  }
  while (t < n) {
    step(s0, std::false_type{}, fbx, fby);
    if (++t >= n) break;
    step(s1, std::false_type{}, fby, fbx);
    ++t;
  }

  g_epilogue<8, 8, F32OUT>(g, acc, smem_raw, wave, lane, w.m0, w.n0, w.split, glu_fwd, nb0);
}

// ------------------------------------------------------------------------------------ smaller tiles
// Lets at most `rem` stages of IPS transfers (rem <= MAX) of this wave stay in flight.
template <int IPS, int MAX>
__device__ __forceinline__ void g_wait_stages(int rem) {
  if constexpr (MAX > 0) {
    if (rem >= MAX) { G_VMCNT(MAX * IPS); return; }
    g_wait_stages<IPS, MAX - 1>(rem);
  } else {
    G_VMCNT(0);
  }
}

// Bound: with few blocks the chain barrier -> LDS reads -> products of one stage (no second block covers it), with many the
// matrix cores and, for 64x64, the 16 KiB a stage takes from L2.  Hence a ring as deep as the LDS allows where a unit has one
// block only (128x128: 4 stages, 0.40 us a stage against 0.60 with 2), two blocks and a ring of two where it has several, and
// 64x64 tiles, or shapes between, for what would leave units idle (which of them: see the plan in gemm_bf16.hip).  Measured against 128x128/256x128 kernels with stages of 32 K, half-line
// transfers and 32x32x16 instructions: 4096x768x4096 36 -> 28 us, 4096x1792x4096 with B transposed 66 -> 51,
// 1792x4096x4096 A transposed 65 -> 58, 528x520x1000 10.3 -> 7, 1024x768x768 8.8 -> 5.3, 1088x1408x12544 62 -> 46.
// Tiles of BM x BN through a ring of S stages, OCC blocks per compute unit.  A stage is worked off in two k-steps of 32; the
// fragments of the next k-step are read while the products of the current one are issued (the second k-step starts with
// the barrier that publishes the next stage and frees this one), and the transfer of stage t+S follows that barrier.
template <int BM, int BN, int S, bool TA, bool TB, bool F32OUT>
__device__ __forceinline__ void g_tile(GemmArgs& g, int bx, unsigned char* smem_raw) {
  constexpr int MT = BM / 32, NT = BN / 32, IA = g_transfers<BM, TA>, IB = g_transfers<BN, !TB>;
  constexpr int BYTES_A = g_bytes<BM, TA>, STAGE = BYTES_A + g_bytes<BN, !TB>;
  GemmTile w;
  if (!g_begin<BM, BN>(g, bx, w)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = w.n, n_full = w.n_full;
  uint32_t voa[IA], vob[IB];
  const bool glu_fwd = !TA && !TB && !F32OUT && g.glu_mode == GLU_FWD;
  const int jump = glu_fwd ? g.glu_f - BN / 2 : 0;  // B panel: BN/2 gate columns, then the up columns of the same outputs
  const int nb0 = glu_fwd ? w.tn * (BN / 2) : w.n0;
  g_offsets<BM, TA>(voa, w.m0, g.M, g.K, wave, lane);
  g_offsets<BN, !TB>(vob, nb0, g.N, g.K, wave, lane, jump);
  const size_t sa = (TA ? (size_t)G_BK * g.M : (size_t)G_BK) * sizeof(bf16_t);
  const size_t sb = (TB ? (size_t)G_BK : (size_t)G_BK * g.N) * sizeof(bf16_t);
  const char* ap = g_uniform(reinterpret_cast<const char*>(g.A + (TA ? (size_t)w.k_begin * g.M + w.m0 : (size_t)w.m0 * g.K + w.k_begin)));
  const char* bp = g_uniform(reinterpret_cast<const char*>(g.B + (TB ? (size_t)nb0 * g.K + w.k_begin : (size_t)w.k_begin * g.N + nb0)));
  const uint32_t lds0 = lds_address(smem_raw), la0 = lds0 + wave * (IA * 1024), lb0 = lds0 + BYTES_A + wave * (IB * 1024);
  g_bias_transfers(ap, voa);
  g_bias_transfers(bp, vob);
  auto issue = [&](int t, uint32_t slot) {  // stage t into the slot at byte offset `slot`
    if (t < n_full) {
      g_transfers_of_stage(la0 + slot, ap, voa);
      g_transfers_of_stage(lb0 + slot, bp, vob);
    } else {
      g_issue_ragged<BM, TA>(la0 + slot, g.A, w.m0, w.k_begin + t * G_BK, g.M, g.K, w.k_end, wave, lane);
      g_issue_ragged<BN, !TB>(lb0 + slot, g.B, nb0, w.k_begin + t * G_BK, g.N, g.K, w.k_end, wave, lane, jump);
    }
    ap += sa;
    bp += sb;
  };
  for (int t = 0; t < S && t < n; t++) issue(t, t * STAGE);
  f32x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; i++)
#pragma unroll
    for (int j = 0; j < NT; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  g_settle(acc);
  const lds_char* pa[4];
  const lds_char* pb[4];
  g_pointers<TA>(pa, (const lds_char*)smem_raw, (wave >> 1) * MT, lane);
  g_pointers<!TB>(pb, (const lds_char*)smem_raw + BYTES_A, (wave & 1) * NT, lane);
  bf16x8 fa[2][MT], fb[2][NT];
  // fragment r of a k-step: A's first, then all of B's (the first products need those), then A's others
  auto read = [&](int ks, int r) {
    if (r == 0) fa[ks][0] = g_frag<TA>(pa, ks, 0);
    else if (r <= NT) fb[ks][r - 1] = g_frag<!TB>(pb, ks, r - 1);
    else fa[ks][r - NT] = g_frag<TA>(pa, ks, r - NT);
  };
  // Spreads COUNT actions over the products [first, first + over): does those that belong to product i.
  auto spread = [](int i, int first, int over, int count, auto act) {
    const int x = i - first;
    if (x < 0 || x >= over) return;
#pragma unroll
    for (int q = 0; q <= count / over; q++) {
      const int a = (x * count + over - 1) / over + q;
      if (a < count && a * over / count == x) act(a);
    }
  };
  // Chained K ranges (see the plan): the sum of a finished range moves to `total` and the next one starts from zero.
  f32x4 total[MT][NT];  // holds nothing before the first range's end
  auto kstep = [&](int ks, auto aux) {
#pragma unroll
    for (int i = 0; i < MT * NT; i++) {
      const int x = i / NT, y = i % NT;
      g_mfma(acc[x][y], fb[ks][y], fa[ks][x]);
      aux(i);
      G_PIN();
    }
  };
  if (n > 0) {
    g_wait_stages<IA + IB, S - 1>(min(S, n) - 1);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < MT + NT; r++) read(0, r);
  }
  int slot = 0;
  auto step = [&](auto steady, int t) {
    constexpr bool STEADY = decltype(steady)::value;
    constexpr int MM = MT * NT, R = MT + NT, D = IA + IB, BI = MM >= 16 ? 3 : 0;
    kstep(0, [&](int i) { spread(i, 0, MM * 3 / 4, R, [&](int r) { read(1, r); }); });
    const int next = slot + STAGE == S * STAGE ? 0 : slot + STAGE;
#pragma unroll
    for (int x = 0; x < 4; x++) {
      pa[x] += next - slot;
      pb[x] += next - slot;
    }
    uint32_t m = 0;
    kstep(1, [&](int i) {
      if (i == BI) {
        if (STEADY) G_VMCNT((S - 2) * D);
        else g_wait_stages<D, S - 2>(min(n - 1, t + S - 1) - (t + 1));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (!STEADY && t + S < n) issue(t + S, slot);
      }
      spread(i, BI, MM - BI, R, [&](int r) { read(0, r); });
      if (STEADY)
        spread(i, BI, MM - BI, D, [&](int d) {
          if (d == 0) m = dma_lds(la0 + slot + G_BIAS);
          if (d == IA) m = dma_lds(lb0 + slot + G_BIAS);
          if (d < IA) dma16_at(m, ap, voa[d], d * 1024 - G_BIAS);
          else dma16_at(m, bp, vob[d - IA], (d - IA) * 1024 - G_BIAS);
        });
    });
    if (STEADY) {
      ap += sa;
      bp += sb;
    }
    slot = next;
  };
  const int range = g.k_chain > 0 ? g.k_chain / G_BK : n;  // stages
  for (int t = 0; t < n;) {
    const int end = min(n, t + range), steady_end = min(end, n_full - S);
    for (; t < steady_end; t++) step(std::true_type{}, t);
    for (; t < end; t++) step(std::false_type{}, t);
    if (t == n) break;
    g_settle(acc);
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) {
        total[i][j] = t == range ? acc[i][j] : total[i][j] + acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    g_settle(acc);
  }
  if (n > range) {
    g_settle(acc);
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) acc[i][j] = total[i][j] + acc[i][j];
  }
  g_epilogue<MT, NT, F32OUT>(g, acc, smem_raw, wave, lane, w.m0, w.n0, w.split, glu_fwd, nb0);
}
template <int BM, int BN, int S, int OCC, bool TA, bool TB, bool F32OUT>
__global__ __launch_bounds__(256, OCC) void gemm_bf16_tile_kernel(GemmArgs g, const GemmAr ar) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  if (g_standin_block(g, ar)) return;
  g_tile<BM, BN, S, TA, TB, F32OUT>(g, (int)blockIdx.x - g.ar_blocks, smem_raw);
}

// A column sum (a bias gradient) that a pair's launch carries: blocks from `first` on, 32 columns each.
struct GemmColsum {
  BiasGrad of;
  int first;
};
// The sums of colsum_direct_kernel in its order, the same bits, by 256 threads in four turns: 256 row lanes add every 256th row, then the
// sixteen lanes of each of sixteen groups, then the groups.
__device__ __forceinline__ void g_colsum(const BiasGrad& c, int blk, float* smem) {
  const int cl = threadIdx.x & 3, col = blk * 32 + cl * 8, colc = min(col, c.n - 8);
#pragma unroll
  for (int p = 0; p < 4; p++) {
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int r = p * 64 + (threadIdx.x >> 2); r < c.rows; r += 256 * 8) {
      bf16x8 v[8];
#pragma unroll
      for (int u = 0; u < 8; u++) v[u] = *reinterpret_cast<const bf16x8*>(c.x + (size_t)min(r + 256 * u, c.rows - 1) * c.n + colc);
#pragma unroll
      for (int u = 0; u < 8; u++)
#pragma unroll
        for (int i = 0; i < 8; i++) s[i] = r + 256 * u < c.rows ? s[i] + (float)v[u][i] : s[i];
    }
#pragma unroll
    for (int d = 4; d < 64; d <<= 1)
#pragma unroll
      for (int i = 0; i < 8; i++) s[i] += __shfl_xor(s[i], d, 64);
    if ((threadIdx.x & 63) < 4)
#pragma unroll
      for (int i = 0; i < 8; i++) smem[(p * 4 + (threadIdx.x >> 6)) * 32 + cl * 8 + i] = s[i];
  }
  __syncthreads();
  if (threadIdx.x < 32 && blk * 32 + (int)threadIdx.x < c.n) {
    float t = smem[threadIdx.x];
#pragma unroll
    for (int k = 1; k < 16; k++) t += smem[k * 32 + threadIdx.x];
    c.dst[blk * 32 + threadIdx.x] += t;
  }
}

// A data gradient (A [M,K], B [N,K], bf16 result) and a weight gradient (A [K,M], B [K,N], added to float32) in one launch: the two
// GEMMs of a linear layer's backward pass read the same dY and do not depend on each other.  The first n_first blocks are
// the tiles of the one whose blocks take longer.
template <int BM, int BN, int S, int OCC>
__global__ __launch_bounds__(256, OCC) void gemm_bf16_pair_kernel(GemmArgs d, GemmArgs w, int n_first, int w_first, const GemmColsum cs) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const bool second = (int)blockIdx.x >= n_first;
  if (__builtin_expect(second && (int)blockIdx.x >= cs.first, 0)) {
    g_colsum(cs.of, (int)blockIdx.x - cs.first, reinterpret_cast<float*>(smem_raw));
    return;
  }
  const int bx = second ? (int)blockIdx.x - n_first : (int)blockIdx.x;
  if (second != (w_first != 0)) g_tile<BM, BN, S, true, false, true>(w, bx, smem_raw);
  else g_tile<BM, BN, S, false, true, false>(d, bx, smem_raw);
}

static int allow_lds(const void* kernel, bool* attr_set, int bytes) {
  const int dev = dh_device_index();
  if (!attr_set[dev]) {  // the attribute belongs to the kernel's code object on one device
    DH_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    attr_set[dev] = true;
  }
  return DH_OK;
}
// A block counts its K ranges in stages: of a range that is no whole number of them it would make another one, of less than a stage none that ends.
static int g_check_chain(const GemmArgs& g) {
  if (g.k_chain < 0 || g.k_chain % G_BK) DH_FAIL(DH_ERR_INVALID_ARG, "gemm: K ranges of %d are no whole stages of %d", g.k_chain, G_BK);
  return DH_OK;
}
// Launches `kernel` (tiles of BM x BN, LDS_BYTES of dynamic LDS) over the launch indices [tile_first, tile_first + n_tiles)
// (n_tiles < 0: all of them).
template <int BM, int BN, int LDS_BYTES, typename Kernel>
static int launch_tiles(Kernel kernel, bool* attr_set, GemmArgs g, int splits, hipStream_t stream, int n_groups, int tile_first, int n_tiles,
                        const GemmAr* ar) {
  int rc = g_check_chain(g);
  if (rc || (rc = allow_lds((const void*)kernel, attr_set, LDS_BYTES))) return rc;
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (g.N + BN - 1) / BN;
  g.n_split = n_tiles < 0 ? splits : 0;
  g.tiles_per_xcd = (g.tiles_m * g.tiles_n * std::max(1, g.n_split) + 7) / 8;
  g.tile_first = tile_first;
  dim3 grid((n_tiles >= 0 ? n_tiles : g.tiles_per_xcd * 8) + g.ar_blocks, g.n_split > 0 ? 1 : splits, n_groups);
  GemmAr none;
  none.ranks = 0; none.n8 = 0; none.out = nullptr;
  for (int r = 0; r < DH_MAX_RANKS; r++) none.parts.p[r] = nullptr;
  kernel<<<grid, 256, LDS_BYTES, stream>>>(g, ar ? *ar : none);
  DH_LAUNCH_CHECK();
  return DH_OK;
}
template <bool TA, bool TB, bool F32OUT>
static int launch_wide(const GemmArgs& g, int splits, hipStream_t stream, int n_groups = 1, int tile_first = 0, int n_tiles = -1,
                       const GemmAr* ar = nullptr) {
  static bool attr_set[DH_MAX_DEVICES] = {};
  return launch_tiles<256, 256, GW_RING * GW_SLOT>(gemm_bf16_wide_kernel<TA, TB, F32OUT>, attr_set, g, splits, stream, n_groups, tile_first, n_tiles, ar);
}
template <int BM, int BN, int S, bool TA, bool TB, bool F32OUT>
constexpr int g_lds_bytes() {  // the ring, or the epilogue's turn of the tile where that takes more
  constexpr int ring = S * (g_bytes<BM, TA> + g_bytes<BN, !TB>), epilogue = F32OUT ? BM * 256 : BM * BN * 2;
  return epilogue > ring ? epilogue : ring;
}
template <int BM, int BN, int S, int OCC, bool TA, bool TB, bool F32OUT>
static int launch_tile(const GemmArgs& g, int splits, hipStream_t stream, int n_groups, int tile_first, int n_tiles, const GemmAr* ar) {
  static bool attr_set[DH_MAX_DEVICES] = {};
  return launch_tiles<BM, BN, g_lds_bytes<BM, BN, S, TA, TB, F32OUT>()>(gemm_bf16_tile_kernel<BM, BN, S, OCC, TA, TB, F32OUT>, attr_set, g, splits, stream, n_groups,
                                                        tile_first, n_tiles, ar);
}

// Launches the tile shape `cfg` (GemmPlan).  Instantiated for each layout and result type in a source of its own.
template <bool TA, bool TB, bool F32OUT>
int launch_out(const GemmArgs& g, int cfg, int splits, hipStream_t stream, int n_groups, int tile_first, int n_tiles, const GemmAr* ar) {
  switch (cfg) {
    case 0: return launch_wide<TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 2: return launch_tile<256, 128, 3, 1, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 3: return launch_tile<64, 64, 4, 2, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 4: return launch_tile<128, 128, 4, 1, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 5: return launch_tile<192, 128, 4, 1, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 6: return launch_tile<96, 128, 4, 1, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 7: return launch_tile<96, 128, 2, 2, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 8: return launch_tile<64, 128, 3, 2, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    default: return launch_tile<128, 128, 2, 2, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
  }
}

template <int BM, int BN, int S, int OCC>
static int launch_pair_tile(GemmArgs d, GemmArgs w, bool w_first, hipStream_t stream, int n_groups, const BiasGrad* bias, bool* carried) {
  static bool attr_set[DH_MAX_DEVICES] = {};
  constexpr int ld = g_lds_bytes<BM, BN, S, false, true, false>(), lw = g_lds_bytes<BM, BN, S, true, false, true>(), lds = ld > lw ? ld : lw;
  int rc;
  if ((rc = g_check_chain(d)) || (rc = g_check_chain(w)) || (rc = allow_lds((const void*)gemm_bf16_pair_kernel<BM, BN, S, OCC>, attr_set, lds))) return rc;
  int blocks[2];
  GemmArgs* g[2] = {&d, &w};
  for (int i = 0; i < 2; i++) {
    g[i]->tiles_m = (g[i]->M + BM - 1) / BM;
    g[i]->tiles_n = (g[i]->N + BN - 1) / BN;
    g[i]->tiles_per_xcd = (g[i]->tiles_m * g[i]->tiles_n + 7) / 8;
    blocks[i] = g[i]->tiles_per_xcd * 8;
  }
  // A column sum of one launch rides along where units are free for its blocks: of the backward chain of a small layer it is a launch of 4 us less per linear
  // (4 heads x 2 x 264 tokens, 520 wide: the step 141 -> 126).  Behind tiles that fill the units it would be a round of its own.
  GemmColsum cs = {{nullptr, 0, 0, nullptr}, blocks[0] + blocks[1]};
  int extra = 0;
  if (bias != nullptr && dh_colsum_direct(bias->rows, bias->n) && cs.first + (bias->n + 31) / 32 <= OCC * d.cus) {
    cs.of = *bias;
    extra = (bias->n + 31) / 32;
    *carried = true;
  }
  gemm_bf16_pair_kernel<BM, BN, S, OCC><<<dim3(cs.first + extra, 1, n_groups), 256, lds, stream>>>(d, w, blocks[w_first ? 1 : 0], w_first ? 1 : 0, cs);
  DH_LAUNCH_CHECK();
  return DH_OK;
}
// Launches the pair with tile shape `cfg`.  Three sources hold the shapes, so that they compile side by side.
template <int CFG>
int launch_pair(const GemmArgs& d, const GemmArgs& w, bool w_first, hipStream_t stream, int n_groups, const BiasGrad* bias, bool* carried) {
  if constexpr (CFG == 2) return launch_pair_tile<256, 128, 3, 1>(d, w, w_first, stream, n_groups, bias, carried);
  else if constexpr (CFG == 3) return launch_pair_tile<64, 64, 4, 2>(d, w, w_first, stream, n_groups, bias, carried);
  else if constexpr (CFG == 4) return launch_pair_tile<128, 128, 4, 1>(d, w, w_first, stream, n_groups, bias, carried);
  else if constexpr (CFG == 5) return launch_pair_tile<192, 128, 4, 1>(d, w, w_first, stream, n_groups, bias, carried);
  else if constexpr (CFG == 6) return launch_pair_tile<96, 128, 4, 1>(d, w, w_first, stream, n_groups, bias, carried);
  else if constexpr (CFG == 7) return launch_pair_tile<96, 128, 2, 2>(d, w, w_first, stream, n_groups, bias, carried);
  else if constexpr (CFG == 8) return launch_pair_tile<64, 128, 3, 2>(d, w, w_first, stream, n_groups, bias, carried);
  else return launch_pair_tile<128, 128, 2, 2>(d, w, w_first, stream, n_groups, bias, carried);
}
