// bf16 GEMM on the matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation.
//   C[M,N] (+)= opA(A) * opB(B)
// Operand layouts (all row-major):
//   TA = false: A is [M,K] (K contiguous)      TA = true: A is [K,M] (M contiguous)
//   TB = false: B is [K,N] (N contiguous)      TB = true: B is [N,K] (K contiguous)
// The forward projections use (TA=0,TB=0) with weights [in,out]; data gradients (dY * W^T) use
// (TA=0,TB=1); weight gradients (X^T * dY) use (TA=1,TB=0) and add into a float32 buffer.
//
// Two kernels: gemm_bf16_wide_kernel (256x256 tiles) takes the products that fill the chip with such tiles,
// gemm_bf16_tile_kernel (256x128 down to 64x64) the smaller ones.  Common to both: a block is four waves in 2x2, one per
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
#include <algorithm>
#include <climits>
#include <type_traits>
#include <utility>
#include "common.h"
#include "dma.h"

#define G_BK 64  // K of a stage

// f(0), f(1), ..., f(N-1) with compile-time arguments
template <typename F, int... I>
__device__ __forceinline__ void static_for_each(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

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
  int k_per_split;   // K handled by one split (a multiple of 32)
  int tiles_m, tiles_n, tiles_per_xcd;
  const bf16_t* bias;          // optional [N], added before the bf16 store
  const int32_t* group_rows;   // grouped GEMM: device array of row counts (blockIdx.z = group), else nullptr
  int group_mode;              // 0/1: groups split M (A and C rows), B per group; 2: groups split K, C per group
  // Modes 0/1 are issued as two launches: part 1 with the large tile, part 2 with the 128x128 tile.  When the groups'
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
  int k_chain;  // 64x64 tiles: K range summed on its own before it joins the total (a multiple of 32; 0: the whole split)
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

// Row of the operand's non-K dimension (relative to the tile of ROWS) and k of the 16-byte chunk lane `lane` fetches in
// transfer j (of ROWS/32) of wave `wave`.
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ void g_chunk(int wave, int j, int lane, int& r, int& k) {
  const int inst = wave * (ROWS / 32) + j;
  if (KMAJOR) {
    k = (inst & 7) * 8 + (lane >> 3);
    const int slot = ((lane & 7) >> 1) ^ (((k >> 1) & 1) | (((k >> 3) & 1) << 1));
    r = (inst >> 3) * 64 + slot * 16 + (lane & 1) * 8;
  } else {
    r = inst * 8 + (lane >> 3);
    k = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
  }
}
// Byte offsets relative to the tile's origin.  half_jump: the tile's second half of columns lies that many columns further on.
template <int ROWS, bool KMAJOR>
__device__ __forceinline__ void g_offsets(uint32_t (&voff)[ROWS / 32], int r0, int R, int K, int wave, int lane, int half_jump = 0) {
#pragma unroll
  for (int j = 0; j < ROWS / 32; j++) {
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
  for (int j = 0; j < ROWS / 32; j++) {
    int r, k;
    g_chunk<ROWS, KMAJOR>(wave, j, lane, r, k);
    r += r0 + (r >= ROWS / 2 ? half_jump : 0);
    k += k0;
    const bf16_t* src = (r < R && k < k_end) ? base + (KMAJOR ? (size_t)k * R + r : (size_t)r * K + k) : reinterpret_cast<const bf16_t*>(dh_zero_chunk);
    dma16(src, lds_wave + j * 1024);
  }
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
    constexpr int PASSES = WM / 8, U = PASSES < 8 ? PASSES : 8, UNITS = PASSES / U;  // 8 rows a pass, U passes a unit
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
      constexpr int PASSES = WM / RPP, NB = PASSES < 8 ? PASSES : 8;
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

// What a block works on: false if it has no tile (it carried a share of the stand-in, or is surplus).
struct GemmTile {
  int m0, n0, tn, split, k_begin, n, n_full, k_end;  // n: stages of its K range, of which the first n_full are whole
};
template <int BM, int BN>
__device__ __forceinline__ bool g_begin(GemmArgs& g, const GemmAr& ar, GemmTile& w) {
  if (g.ar_blocks > 0 && blockIdx.x < (unsigned)g.ar_blocks) {  // this block is a share of the stand-in, not a tile
    if (blockIdx.y == 0 && blockIdx.z == 0)
      allreduce_span<bf16_t>(ar.parts, ar.ranks, ar.out, ar.n8, (size_t)blockIdx.x * blockDim.x + threadIdx.x,
                             (size_t)g.ar_blocks * blockDim.x);
    return false;
  }
  if (g.group_rows != nullptr && !group_setup<BM>(g)) return false;
  int tm;
  w.split = blockIdx.y;
  if (g.n_split > 1) {  // contiguous ranges again: an XCD works on neighbouring tiles of the same K range
    const int n = g.tiles_m * g.tiles_n, logical = (blockIdx.x & 7) * g.tiles_per_xcd + (blockIdx.x >> 3);
    w.split = __builtin_amdgcn_readfirstlane(logical / n);
    if (w.split >= g.n_split) return false;
    tile_of_logical(logical - w.split * n, g.tiles_m, g.tiles_n, tm, w.tn);
  } else if (!tile_of_launch((int)blockIdx.x - g.ar_blocks + g.tile_first, g.tiles_m, g.tiles_n, g.tiles_per_xcd, tm, w.tn)) {
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
// K is consumed 64 at a time from two LDS stages (A and B, 32 KiB each).  A K tile is worked off in four quadrants
// (a0 b0, a0 b1, a1 b1, a1 b0: halves of 64 rows / columns); the fragments of the half that comes next are read while
// the current quadrant's products are issued, so a stage has been read completely after the second quadrant.  One barrier
// there (it also publishes the next stage), and the transfers of tile t+2 follow into the stage just emptied.  Matrix
// instructions, LDS reads and transfers are interleaved two products at a time and pinned in that order.
#define GW_STAGE 65536u

template <bool TA, bool TB, bool F32OUT>
__global__ __launch_bounds__(256, 1) void gemm_bf16_wide_kernel(GemmArgs g, const GemmAr ar) {
  GemmTile w;
  if (!g_begin<256, 256>(g, ar, w)) return;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool glu_fwd = !TA && !TB && !F32OUT && g.glu_mode == GLU_FWD;
  const int jump = glu_fwd ? g.glu_f - 128 : 0;  // B panel: 128 gate columns, then the 128 up columns of the same outputs
  const int nb0 = glu_fwd ? w.tn * 128 : w.n0, n = w.n, n_full = w.n_full;

  uint32_t voa[8], vob[8];
  g_offsets<256, TA>(voa, w.m0, g.M, g.K, wave, lane);
  g_offsets<256, !TB>(vob, nb0, g.N, g.K, wave, lane, jump);
  const size_t sa = (TA ? (size_t)G_BK * g.M : (size_t)G_BK) * sizeof(bf16_t);
  const size_t sb = (TB ? (size_t)G_BK : (size_t)G_BK * g.N) * sizeof(bf16_t);
  // next tile to transfer
  const char* ap = g_uniform(reinterpret_cast<const char*>(g.A + (TA ? (size_t)w.k_begin * g.M + w.m0 : (size_t)w.m0 * g.K + w.k_begin)));
  const char* bp = g_uniform(reinterpret_cast<const char*>(g.B + (TB ? (size_t)nb0 * g.K + w.k_begin : (size_t)w.k_begin * g.N + nb0)));
  const uint32_t ldsA = lds_address(smem_raw) + wave * 8192u, ldsB = ldsA + 32768u;
  auto issue = [&](int t) {
    const uint32_t so = (t & 1) * GW_STAGE;
    if (t < n_full) {
#pragma unroll
      for (int j = 0; j < 8; j++) dma16_base(ap, voa[j], ldsA + so + j * 1024);
#pragma unroll
      for (int j = 0; j < 8; j++) dma16_base(bp, vob[j], ldsB + so + j * 1024);
    } else {
      g_issue_ragged<256, TA>(ldsA + so, g.A, w.m0, w.k_begin + t * G_BK, g.M, g.K, w.k_end, wave, lane);
      g_issue_ragged<256, !TB>(ldsB + so, g.B, nb0, w.k_begin + t * G_BK, g.N, g.K, w.k_end, wave, lane, jump);
    }
  };
  if (n > 0) issue(0);
  ap += sa;
  bp += sb;
  if (n > 1) issue(1);
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
  g_pointers<TA>(pa, (const lds_char*)smem_raw, (wave >> 1) * 8, lane);
  g_pointers<!TB>(pb, (const lds_char*)smem_raw + 32768, (wave & 1) * 8, lane);

  bf16x8 fa0[8], fa1[8], fbx[8], fby[8];  // halves of 64 rows / columns: [k-step of 32][16-row tile]
  auto rd_a = [&](int half, int e) { return g_frag<TA>(pa, e >> 2, half * 4 + (e & 3)); };
  auto rd_b = [&](int half, int e) { return g_frag<!TB>(pb, e >> 2, half * 4 + (e & 3)); };
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
  if (n > 0) {
    if (n > 1) G_VMCNT(16); else G_VMCNT(0);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; e++) { fa0[e] = rd_a(0, e); fbx[e] = rd_b(0, e); }
  }
  int t = 0;
  // Works off tile t in stage S.  b0 holds the fragments of its first B half, b1 receives those of the second and then
  // the next tile's first half.  STEADY: tile t+2 is a full tile, its transfers go out between the products.
  auto step = [&](auto stage, auto steady, bf16x8 (&f0)[8], bf16x8 (&f1)[8]) {
    constexpr int S = decltype(stage)::value;
    constexpr bool STEADY = decltype(steady)::value;
    constexpr int to_next = S == 0 ? (int)GW_STAGE : -(int)GW_STAGE;
    quad(fa0, f0, 0, 0, [&](int i) { if ((i & 1) == 0) f1[i >> 1] = rd_b(1, i >> 1); });
    quad(fa0, f1, 0, 1, [&](int i) {
      if (i < 8) fa1[i] = rd_a(1, i);
      if (i == 13) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    });
    shift(pa, to_next);
    shift(pb, to_next);
    if (!STEADY && t + 2 < n) issue(t + 2);
    quad(fa1, f1, 1, 1, [&](int i) {
      if ((i & 1) == 0) fa0[i >> 1] = rd_a(0, i >> 1);
      else if (STEADY) dma16_base(ap, voa[i >> 1], ldsA + S * GW_STAGE + (i >> 1) * 1024);
    });
    quad(fa1, f0, 1, 0, [&](int i) {
      if ((i & 1) == 0) f1[i >> 1] = rd_b(0, i >> 1);
      else if (STEADY) dma16_base(bp, vob[i >> 1], ldsB + S * GW_STAGE + (i >> 1) * 1024);
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
// 64x64 tiles for what would leave units idle.  Measured against 128x128/256x128 kernels with stages of 32 K, half-line
// transfers and 32x32x16 instructions: 4096x768x4096 36 -> 28 us, 4096x1792x4096 with B transposed 66 -> 51,
// 1792x4096x4096 A transposed 65 -> 58, 528x520x1000 10.3 -> 7, 1024x768x768 8.8 -> 5.3, 1088x1408x12544 62 -> 46.
// Tiles of BM x BN through a ring of S stages, OCC blocks per compute unit.  A stage is worked off in two k-steps of 32; the
// fragments of the next k-step are read while the products of the current one are issued (the second k-step starts with
// the barrier that publishes the next stage and frees this one), and the transfer of stage t+S follows that barrier.
template <int BM, int BN, int S, int OCC, bool TA, bool TB, bool F32OUT>
__global__ __launch_bounds__(256, OCC) void gemm_bf16_tile_kernel(GemmArgs g, const GemmAr ar) {
  constexpr int MT = BM / 32, NT = BN / 32, IA = BM / 32, IB = BN / 32, STAGE = (BM + BN) * G_BK * 2;
  GemmTile w;
  if (!g_begin<BM, BN>(g, ar, w)) return;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
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
  const uint32_t lds0 = lds_address(smem_raw), la0 = lds0 + wave * (IA * 1024), lb0 = lds0 + BM * 128 + wave * (IB * 1024);
  auto issue = [&](int t, uint32_t slot) {  // stage t into the slot at byte offset `slot`
    if (t < n_full) {
#pragma unroll
      for (int j = 0; j < IA; j++) dma16_base(ap, voa[j], la0 + slot + j * 1024);
#pragma unroll
      for (int j = 0; j < IB; j++) dma16_base(bp, vob[j], lb0 + slot + j * 1024);
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
  g_pointers<!TB>(pb, (const lds_char*)smem_raw + BM * 128, (wave & 1) * NT, lane);
  bf16x8 fa[2][MT], fb[2][NT];
  // fragment r of a k-step: A's first, then all of B's (the first products need those), then A's others
  auto read = [&](auto ks, auto r) {
    if constexpr (r == 0) fa[ks][0] = g_frag<TA>(pa, ks, 0);
    else if constexpr (r <= NT) fb[ks][r - 1] = g_frag<!TB>(pb, ks, r - 1);
    else fa[ks][r - NT] = g_frag<TA>(pa, ks, r - NT);
  };
  // Chained K ranges (see the plan): the sum of a finished range moves to `total` and the next one starts from zero.
  constexpr bool CHAIN = BM == 64 && BN == 64;
  f32x4 total[CHAIN ? MT : 1][CHAIN ? NT : 1];
  const int range_steps = g.k_chain > 0 ? g.k_chain / 32 : INT_MAX;
  int to_flush = range_steps;  // k-steps left in the range
  if constexpr (CHAIN) {
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) total[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto range_end = [&] {
    if constexpr (CHAIN) {
      if (--to_flush == 0) {
        to_flush = range_steps;
        g_settle(acc);
#pragma unroll
        for (int i = 0; i < MT; i++)
#pragma unroll
          for (int j = 0; j < NT; j++) {
            total[i][j] += acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        g_settle(acc);
      }
    }
  };
  const std::integral_constant<int, 0> k0{};
  const std::integral_constant<int, 1> k1{};
  auto kstep = [&](auto ks, auto aux) {
    static_for<MT * NT>([&](auto i) {
      g_mfma(acc[i / NT][i % NT], fb[ks][i % NT], fa[ks][i / NT]);
      aux(i);
      G_PIN();
    });
  };
  if (n > 0) {
    g_wait_stages<IA + IB, S - 1>(min(S, n) - 1);
    __syncthreads();
    static_for<MT + NT>([&](auto r) { read(k0, r); });
  }
  int slot = 0;
  auto step = [&](auto steady, int t) {
    constexpr bool STEADY = decltype(steady)::value;
    constexpr int MM = MT * NT, R = MT + NT, D = IA + IB, BI = MM >= 16 ? 3 : 0;
    kstep(k0, [&](auto i) {
      static_for<R>([&](auto r) {
        if constexpr (r * (MM * 3 / 4) / R == i) read(k1, r);
      });
    });
    range_end();
    const int next = slot + STAGE == S * STAGE ? 0 : slot + STAGE;
#pragma unroll
    for (int x = 0; x < 4; x++) {
      pa[x] += next - slot;
      pb[x] += next - slot;
    }
    kstep(k1, [&](auto i) {
      if constexpr (i == BI) {
        if (STEADY) G_VMCNT((S - 2) * D);
        else g_wait_stages<D, S - 2>(min(n - 1, t + S - 1) - (t + 1));
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (!STEADY && t + S < n) issue(t + S, slot);
      }
      static_for<R>([&](auto r) {
        if constexpr (BI + r * (MM - BI) / R == i) read(k0, r);
      });
      if constexpr (STEADY)
        static_for<D>([&](auto d) {
          if constexpr (BI + d * (MM - BI) / D == i) {
            if constexpr (d < IA) dma16_base(ap, voa[d], la0 + slot + d * 1024);
            else dma16_base(bp, vob[d - IA], lb0 + slot + (d - IA) * 1024);
          }
        });
    });
    if (STEADY) {
      ap += sa;
      bp += sb;
    }
    slot = next;
    range_end();
  };
  int t = 0;
  for (; t + S < n_full; t++) step(std::true_type{}, t);
  for (; t < n; t++) step(std::false_type{}, t);
  if constexpr (CHAIN) {
    g_settle(acc);
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) acc[i][j] = total[i][j] + acc[i][j];
  }
  g_epilogue<MT, NT, F32OUT>(g, acc, smem_raw, wave, lane, w.m0, w.n0, w.split, glu_fwd, nb0);
}

// Adds the split-K partials in split order; writes bf16 or accumulates into float32.
__global__ void splitk_reduce_kernel(const float* __restrict__ part, int splits, size_t mn, void* __restrict__ C, int epi,
                                     const bf16_t* __restrict__ bias, int N) {
  size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (i >= mn) return;
  f32x4 s = *reinterpret_cast<const f32x4*>(part + i);
  for (int z = 1; z < splits; z++) s += *reinterpret_cast<const f32x4*>(part + (size_t)z * mn + i);
  if (epi == EPI_STORE_BF16) {
    if (bias != nullptr) {
      const bf16x4 bb = *reinterpret_cast<const bf16x4*>(bias + i % N);
      s += f32x4{(float)bb[0], (float)bb[1], (float)bb[2], (float)bb[3]};
    }
    bf16x4 o = {(bf16_t)s[0], (bf16_t)s[1], (bf16_t)s[2], (bf16_t)s[3]};
    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(C) + i) = o;
  } else {
    f32x4* c = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(C) + i);
    *c = *c + s;
  }
}

// Adds the tail tiles' K splits in split order and applies the final epilogue.  grid (BM*BN/4/256, tail tiles).
template <int BM, int BN>
__global__ __launch_bounds__(256) void tail_reduce_kernel(const float* __restrict__ part, int splits, GemmArgs g, int final_epi) {
  int tm, tn;
  if (!tile_of_launch((int)blockIdx.y + g.tile_first, g.tiles_m, g.tiles_n, g.tiles_per_xcd, tm, tn)) return;
  const int e = (blockIdx.x * 256 + threadIdx.x) * 4, r = e / BN, c = e % BN;
  const int row = tm * BM + r, col = tn * BN + c;
  if (row >= g.M || col >= g.N) return;
  const size_t tile_elems = (size_t)BM * BN, n_tail = gridDim.y;
  f32x4 s = *reinterpret_cast<const f32x4*>(part + blockIdx.y * tile_elems + e);
  for (int z = 1; z < splits; z++) s += *reinterpret_cast<const f32x4*>(part + ((size_t)z * n_tail + blockIdx.y) * tile_elems + e);
  const size_t o = (size_t)row * g.N + col;
  if (final_epi == EPI_STORE_BF16) {
    if (g.bias != nullptr) {
      const bf16x4 bb = *reinterpret_cast<const bf16x4*>(g.bias + col);
      s += f32x4{(float)bb[0], (float)bb[1], (float)bb[2], (float)bb[3]};
    }
    bf16x4 b = {(bf16_t)s[0], (bf16_t)s[1], (bf16_t)s[2], (bf16_t)s[3]};
    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16_t*>(g.C) + o) = b;
  } else {
    f32x4* p = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + o);
    *p = *p + s;
  }
}

// ------------------------------------------------------------------------------------ host side
struct GemmPlan {
  int cfg;  // 0: 256x256, 1: 128x128 two blocks a unit, 2: 256x128, 3: 64x64, 4: 128x128 one block a unit
  int bm, bn, ranges, splits, k_per_split;
  int k_chain;                          // 64x64 with the K ranges summed in the block (0: not)
  int tail_tiles, tail_splits, tail_k;  // tail launch (0 tiles = none): its tiles, K splits and K per split
};

static int num_cus() {  // of the current device
  static int cached[DH_MAX_DEVICES] = {};
  const int dev = dh_device_index();
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) cached[dev] = n;
    else cached[dev] = 256;
    (void)hipGetLastError();
  }
  return cached[dev];
}

// What a block of a tile shape takes alone on its unit, in ns: a stage of 64 K, and filling its ring.  Measured on full and
// part-filled chips (4096x3584x4096, 1792x4096x4096, 4096x768x4096, 1024x768x768 in all three layouts).
struct TileCost { int cfg, bm, bn, stage, fill; };
static const TileCost kTiles[] = {{0, 256, 256, 1250, 1500}, {2, 256, 128, 780, 1200}, {4, 128, 128, 400, 800}, {3, 64, 64, 165, 600}};

// K ranges, tile shape, split-K.
//
// The ranges of K that are summed apart (and then added in order) depend on the shape alone (but for the tail's, below), so
// that a product has the same bits whatever tile it is computed with: a product whose tiles (256x256 from 128 of them on, else 256x128 if these
// make one nearly full round, else 128x128) leave a quarter of the units idle has its K cut into as many ranges as
// fill them, of at least 512; with more than one round of 256x256 tiles and a last round at most half full, the tiles of
// that round have theirs cut (the tail, issued apart: it takes 1/splits of a round and a small ordered sum; into fewer ranges,
// or none, where the caller's workspace does not hold them all, so that its bits depend on the workspace too).
//
// The tile shape is the one with the least rounds * (stages * stage + fill + store): large tiles cost least per product, small ones
// leave fewer units idle.  The store goes at a unit's share of the memory's rate, 20 bytes a ns.  Ranges go to blocks of their
// own and through the workspace (splitk_reduce_kernel), or, with 64x64 tiles, are summed one after the other in the block (no workspace, no second launch), whichever is expected sooner.
//
// groups > 0: a grouped launch, `groups` products of this (average) size.  Its K is never cut (a group's extents are known on
// the device alone), so there are no ranges, and every tile shape is considered over the tiles of all groups.
static GemmPlan choose_plan(int M, int N, int K, bool acc, size_t ws_bytes, int groups = 0) {
  const int cus = num_cus();
  auto tiles = [&](int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const int nkt = std::max(1, (K + 31) / 32);  // ranges are made in units of 32
  GemmPlan p = {};
  const long long t256 = tiles(256, 256), t2 = tiles(256, 128);
  const bool wide = t256 * 2 >= cus;
  const long long t = wide ? t256 : (t2 <= cus && t2 * 4 >= (long long)cus * 3) ? t2 : tiles(128, 128);
  int ranges = 1;
  if (groups == 0 && t * 4 <= cus * 3 && nkt >= 32) ranges = std::max(1, std::min((int)(cus / t), nkt / 16));
  const int per = (nkt + ranges - 1) / ranges;
  ranges = (nkt + per - 1) / per;
  p.ranges = ranges;
  const int tail = (int)(t % cus);
  if (wide && t > cus && tail > 0 && tail * 2 <= cus && nkt >= 64 && groups == 0) {
    int ts = std::min(std::min(cus / tail, 8), nkt / 16);
    const size_t bytes = (size_t)(tail + 7) * 256 * 256 * sizeof(float);  // the launch index range is padded to a multiple of 8
    if (ws_bytes / bytes < (size_t)ts) ts = (int)(ws_bytes / bytes);
    if (ts >= 2) {
      const int kt = (nkt + ts - 1) / ts;
      p.cfg = 0; p.bm = p.bn = 256;
      p.splits = 1; p.k_per_split = nkt * 32;
      p.tail_tiles = tail; p.tail_k = kt * 32; p.tail_splits = (nkt + kt - 1) / kt;
      return p;
    }
  }
  const size_t mn = (size_t)M * N;
  double best = 0;
  auto consider = [&](const TileCost& c, int splits, bool chained) {
    const long long blocks = tiles(c.bm, c.bn) * splits * std::max(1, groups);
    const int stages = ((splits > 1 ? per : nkt) + 1) / 2;
    double stage = c.stage, store = (double)c.bm * c.bn * (splits > 1 ? 4 : acc ? 8 : 2) / 20;
    if (c.cfg == 3) stage += chained ? 25 : 0;
    if (c.cfg == 3 && blocks > cus) stage = 230;      // two on a unit: its L2 traffic
    if (c.cfg == 4 && blocks > cus) stage = 430, store *= 0.6;  // two on a unit: a ring of two; one stores while the other multiplies
    double ns = (double)((blocks + cus - 1) / cus) * (stages * stage + c.fill + store);
    if (splits > 1) ns += 4000 + (double)mn * (4 * splits + (acc ? 8 : 2)) / 5000;  // second launch: the partials read at 5 TB/s
    if (best != 0 && ns >= best) return;
    best = ns;
    p.cfg = c.cfg == 4 && blocks > cus ? 1 : c.cfg;  // deeper ring for a unit's only block, else two blocks a unit
    p.bm = c.bm; p.bn = c.bn;
    p.splits = splits;
    p.k_per_split = splits > 1 ? per * 32 : nkt * 32;
    p.k_chain = chained ? per * 32 : 0;
  };
  for (const TileCost& c : kTiles) {
    if (ranges == 1) consider(c, 1, false);
    else if (ws_bytes / (mn * sizeof(float)) >= (size_t)ranges) consider(c, ranges, false);
    if (ranges > 1 && c.cfg == 3) consider(c, 1, true);
  }
  return p;
}

// Launch indices of the tail launch: from the first index of the last round to the end of the (padded) index range.
static void tail_range(int M, int N, const GemmPlan& p, int& first, int& count) {
  const long long t = (long long)((M + p.bm - 1) / p.bm) * ((N + p.bn - 1) / p.bn);
  first = (int)(t / num_cus()) * num_cus();
  count = (int)((t + 7) / 8 * 8) - first;
}

size_t dh_gemm_bf16_ws_bytes(bool ta, bool tb, int M, int N, int K) {
  (void)tb;
  const GemmPlan p = choose_plan(M, N, K, false, (size_t)-1);
  if (p.tail_tiles > 0) {
    int first, count;
    tail_range(M, N, p, first, count);
    return (size_t)count * p.tail_splits * p.bm * p.bn * sizeof(float);
  }
  return p.ranges > 1 ? (size_t)p.ranges * M * N * sizeof(float) : 0;  // whether it is used depends on the result's type, too
}

// Launches `kernel` (tiles of BM x BN, LDS_BYTES of dynamic LDS) over the launch indices [tile_first, tile_first + n_tiles)
// (n_tiles < 0: all of them).
template <int BM, int BN, int LDS_BYTES, typename Kernel>
static int launch_tiles(Kernel kernel, bool* attr_set, GemmArgs g, int splits, hipStream_t stream, int n_groups, int tile_first, int n_tiles,
                        const GemmAr* ar) {
  const int dev = dh_device_index();
  if (!attr_set[dev]) {  // the attribute belongs to the kernel's code object on one device
    DH_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES));
    attr_set[dev] = true;
  }
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
  return launch_tiles<256, 256, 2 * GW_STAGE>(gemm_bf16_wide_kernel<TA, TB, F32OUT>, attr_set, g, splits, stream, n_groups, tile_first, n_tiles, ar);
}
template <int BM, int BN, int S, int OCC, bool TA, bool TB, bool F32OUT>
static int launch_tile(const GemmArgs& g, int splits, hipStream_t stream, int n_groups, int tile_first, int n_tiles, const GemmAr* ar) {
  static bool attr_set[DH_MAX_DEVICES] = {};
  return launch_tiles<BM, BN, S * (BM + BN) * G_BK * 2>(gemm_bf16_tile_kernel<BM, BN, S, OCC, TA, TB, F32OUT>, attr_set, g, splits, stream, n_groups,
                                                        tile_first, n_tiles, ar);
}

template <bool TA, bool TB, bool F32OUT>
static int launch_out(const GemmArgs& g, int cfg, int splits, hipStream_t stream, int n_groups, int tile_first, int n_tiles, const GemmAr* ar) {
  switch (cfg) {
    case 0: return launch_wide<TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 2: return launch_tile<256, 128, 3, 1, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 3: return launch_tile<64, 64, 4, 2, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    case 4: return launch_tile<128, 128, 4, 1, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
    default: return launch_tile<128, 128, 2, 2, TA, TB, F32OUT>(g, splits, stream, n_groups, tile_first, n_tiles, ar);
  }
}
template <bool TA, bool TB>
static int launch_layout(const GemmArgs& g, const GemmPlan& p, hipStream_t stream, int n_groups = 1, int tile_first = 0,
                         int n_tiles = -1, int splits = 0, const GemmAr* ar = nullptr) {
  if (splits == 0) splits = p.splits;
  return g.epi == EPI_STORE_BF16 ? launch_out<TA, TB, false>(g, p.cfg, splits, stream, n_groups, tile_first, n_tiles, ar)
                                 : launch_out<TA, TB, true>(g, p.cfg, splits, stream, n_groups, tile_first, n_tiles, ar);
}
template <typename... Args>
static int launch_any(bool ta, bool tb, Args... args) {
  if (!ta && !tb) return launch_layout<false, false>(args...);
  if (!ta && tb) return launch_layout<false, true>(args...);
  return launch_layout<true, false>(args...);
}

int dh_launch_gemm_bf16(bool ta, bool tb, int M, int N, int K, const bf16_t* A, const bf16_t* B, void* C,
                        bool out_f32_accumulate, const bf16_t* bias, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (M < 0 || N < 0 || K < 0) DH_FAIL(DH_ERR_SHAPE, "gemm: negative dimension");
  if (N % 8 || (ta ? M : K) % 8 || (tb ? K : N) % 8)
    DH_FAIL(DH_ERR_SHAPE, "gemm (bf16): N and the contiguous operand dimensions must be multiples of 8 (M=%d N=%d K=%d ta=%d tb=%d)", M, N, K, ta, tb);
  if (ta && tb) DH_FAIL(DH_ERR_UNSUPPORTED, "gemm (bf16): trans_a with trans_b is not used by the layer and not built");
  if (bias && out_f32_accumulate) DH_FAIL(DH_ERR_INVALID_ARG, "gemm (bf16): a bias goes with a bf16 result only");
  if (M == 0 || N == 0) return DH_OK;
  if ((long long)M * N >= (1ll << 40) || (long long)M * K >= (1ll << 40)) DH_FAIL(DH_ERR_SHAPE, "gemm: matrix too large");
  GemmPlan p = choose_plan(M, N, K, out_f32_accumulate, ws ? ws_bytes : 0);
  GemmArgs g;
  g.M = M; g.N = N; g.K = K; g.A = A; g.B = B;
  g.k_per_split = p.k_per_split; g.k_chain = p.k_chain; g.n_split = 0;
  g.tiles_m = g.tiles_n = g.tiles_per_xcd = 0;
  g.bias = bias; g.group_rows = nullptr; g.group_mode = 0;
  g.group_part = 0; g.n_groups = 1; g.part1_bm = g.part1_bn = 256; g.cus = 0; g.tile_first = 0;
  g.glu_mode = GLU_NONE; g.glu_f = 0; g.glu_in = nullptr; g.glu_out = nullptr; g.ar_blocks = 0;
  const int final_epi = out_f32_accumulate ? EPI_ACC_F32 : EPI_STORE_BF16;
  int rc;
  if (p.tail_tiles > 0) {  // whole rounds with the final epilogue, then the last round's tiles with K split, then their sum
    int first, count;
    tail_range(M, N, p, first, count);
    g.C = C; g.epi = final_epi;
    if ((rc = launch_any(ta, tb, g, p, stream, 1, 0, first, 1))) return rc;
    GemmArgs gt = g;
    gt.C = ws; gt.epi = EPI_TAIL_F32; gt.k_per_split = p.tail_k;
    if ((rc = launch_any(ta, tb, gt, p, stream, 1, first, count, p.tail_splits))) return rc;
    gt.C = C;
    gt.tiles_m = (M + p.bm - 1) / p.bm; gt.tiles_n = (N + p.bn - 1) / p.bn;
    gt.tiles_per_xcd = (gt.tiles_m * gt.tiles_n + 7) / 8;
    gt.tile_first = first;
    tail_reduce_kernel<256, 256><<<dim3(256 * 256 / 4 / 256, count), 256, 0, stream>>>((const float*)ws, p.tail_splits, gt, final_epi);
    DH_LAUNCH_CHECK();
    return DH_OK;
  }
  if (p.splits > 1) { g.C = ws; g.epi = EPI_PARTIAL_F32; } else { g.C = C; g.epi = final_epi; }
  if ((rc = launch_any(ta, tb, g, p, stream))) return rc;
  if (p.splits > 1) {
    const size_t mn = (size_t)M * N;  // multiple of 8 because N is
    splitk_reduce_kernel<<<(unsigned)((mn / 4 + 255) / 256), 256, 0, stream>>>((const float*)ws, p.splits, mn, C, final_epi, bias, N);
    DH_LAUNCH_CHECK();
  }
  return DH_OK;
}

// GEMM with an all-reduce stand-in in the same launch.  ar_blocks counts 256-thread blocks, as dh_comm_standin's
// n_blocks does.
bool dh_gemm_ar_fits(bool ta, bool tb, int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0 || (ta && tb) || N % 8 || (ta ? M : K) % 8 || (tb ? K : N) % 8) return false;
  const GemmPlan p = choose_plan(M, N, K, false, (size_t)-1);
  return p.splits == 1 && p.tail_tiles == 0;
}
int dh_launch_gemm_bf16_ar(bool ta, bool tb, int M, int N, int K, const bf16_t* A, const bf16_t* B, void* C, bool out_f32_accumulate,
                           int n_ranks, const void* const* parts, bf16_t* ar_out, size_t ar_elems, int ar_blocks, hipStream_t stream) {
  if (!dh_gemm_ar_fits(ta, tb, M, N, K)) DH_FAIL(DH_ERR_UNSUPPORTED, "gemm+allreduce: M=%d N=%d K=%d does not run as a single launch", M, N, K);
  if (n_ranks < 1 || n_ranks > DH_MAX_RANKS || ar_blocks < 1 || ar_blocks > 65536 || ar_elems % 8 || ar_elems == 0)
    DH_FAIL(DH_ERR_INVALID_ARG, "gemm+allreduce: n_ranks %d, n_blocks %d, elements %zu", n_ranks, ar_blocks, ar_elems);
  const GemmPlan p = choose_plan(M, N, K, false, (size_t)-1);
  GemmArgs g;
  g.M = M; g.N = N; g.K = K; g.A = A; g.B = B; g.C = C;
  g.epi = out_f32_accumulate ? EPI_ACC_F32 : EPI_STORE_BF16;
  g.k_per_split = p.k_per_split; g.k_chain = p.k_chain; g.n_split = 0;
  g.tiles_m = g.tiles_n = g.tiles_per_xcd = 0;
  g.bias = nullptr; g.group_rows = nullptr; g.group_mode = 0;
  g.group_part = 0; g.n_groups = 1; g.part1_bm = g.part1_bn = 256; g.cus = 0; g.tile_first = 0;
  g.glu_mode = GLU_NONE; g.glu_f = 0; g.glu_in = nullptr; g.glu_out = nullptr;
  const size_t n8 = ar_elems / 8, want = (n8 + 255) / 256;
  size_t nb = ar_blocks;
  if (nb > want) nb = want;
  g.ar_blocks = (int)nb;
  GemmAr ar;
  ar.ranks = n_ranks; ar.n8 = n8; ar.out = ar_out;
  for (int r = 0; r < DH_MAX_RANKS; r++) ar.parts.p[r] = r < n_ranks ? parts[r] : nullptr;
  return launch_any(ta, tb, g, p, stream, 1, 0, -1, 0, (const GemmAr*)&ar);
}

// Gate/up projection with SwiGLU in its epilogue: gu[T, 2F] = x[T, H] * Wgu[H, 2F] (columns [gate | up]) and
// a[T, F] = gate * sigmoid(gate) * up computed from the stored (rounded) values -- the same bits as
// dh_launch_gemm_bf16 followed by the row-wise kernel.  Fits when the plain GEMM would be one launch and F is a multiple of
// 128 (half the columns of any tile).
bool dh_glu_fwd_fits(int T, int F, int H) {
  if (T <= 0 || F <= 0 || H <= 0 || F % 128 || H % 8) return false;
  const GemmPlan p = choose_plan(T, 2 * F, H, false, (size_t)-1);
  return p.splits == 1 && p.tail_tiles == 0;
}
int dh_launch_gemm_swiglu_fwd_bf16(int T, int F, int H, const bf16_t* x, const bf16_t* Wgu, bf16_t* gu, bf16_t* a, hipStream_t stream) {
  if (!dh_glu_fwd_fits(T, F, H)) DH_FAIL(DH_ERR_SHAPE, "gemm+swiglu forward: T=%d F=%d H=%d does not fit the fused kernel", T, F, H);
  const GemmPlan p = choose_plan(T, 2 * F, H, false, (size_t)-1);
  GemmArgs g;
  g.M = T; g.N = 2 * F; g.K = H; g.A = x; g.B = Wgu; g.C = gu; g.epi = EPI_STORE_BF16;
  g.k_per_split = p.k_per_split; g.k_chain = p.k_chain; g.n_split = 0;
  g.tiles_m = g.tiles_n = g.tiles_per_xcd = 0;
  g.bias = nullptr; g.group_rows = nullptr; g.group_mode = 0;
  g.group_part = 0; g.n_groups = 1; g.part1_bm = g.part1_bn = 256; g.cus = 0; g.tile_first = 0;
  g.glu_mode = GLU_FWD; g.glu_f = F; g.glu_in = nullptr; g.glu_out = a; g.ar_blocks = 0;
  return launch_layout<false, false>(g, p, stream);
}

// Data gradient of the down projection with SwiGLU's backward in its epilogue: dA = dY[T, H] * Wd[F, H]^T is not
// stored; dgu[T, 2F] = (d gate | d up) from dA (rounded to bf16 as the stored dA would be) and gu[T, 2F] -- the same
// bits as the GEMM followed by the row-wise kernel.  Fits when the plain GEMM would be one launch.
bool dh_glu_bwd_fits(int T, int F, int H) {
  if (T <= 0 || F <= 0 || H <= 0 || F % 8 || H % 8) return false;
  const GemmPlan p = choose_plan(T, F, H, false, (size_t)-1);
  return p.splits == 1 && p.tail_tiles == 0;
}
int dh_launch_gemm_swiglu_bwd_bf16(int T, int F, int H, const bf16_t* dy, const bf16_t* Wd, const bf16_t* gu, bf16_t* dgu, hipStream_t stream) {
  if (!dh_glu_bwd_fits(T, F, H)) DH_FAIL(DH_ERR_SHAPE, "gemm+swiglu backward: T=%d F=%d H=%d does not fit the fused kernel", T, F, H);
  const GemmPlan p = choose_plan(T, F, H, false, (size_t)-1);
  GemmArgs g;
  g.M = T; g.N = F; g.K = H; g.A = dy; g.B = Wd; g.C = dgu; g.epi = EPI_STORE_BF16;
  g.k_per_split = p.k_per_split; g.k_chain = p.k_chain; g.n_split = 0;
  g.tiles_m = g.tiles_n = g.tiles_per_xcd = 0;
  g.bias = nullptr; g.group_rows = nullptr; g.group_mode = 0;
  g.group_part = 0; g.n_groups = 1; g.part1_bm = g.part1_bn = 256; g.cus = 0; g.tile_first = 0;
  g.glu_mode = GLU_BWD; g.glu_f = F; g.glu_in = gu; g.glu_out = nullptr; g.ar_blocks = 0;
  return launch_layout<false, true>(g, p, stream);
}

// Grouped GEMM with device-side row counts (expert routing is data): group z owns group_rows[z] consecutive
// rows, max_rows bounds any group (the grid is sized for it).  mode 0: C[rows,dim_b] = A[rows,dim_a] B_z[dim_a,dim_b];
// mode 1: C[rows,dim_b] = A[rows,dim_a] B_z[dim_b,dim_a]^T; mode 2: C_z[dim_a,dim_b] += A[rows,dim_a]^T B[rows,dim_b]
// (float32).  No split-K: every group is one launch slice of the same grid.
static GemmPlan grouped_plan(int mode, int n_groups, int max_rows, int dim_a, int dim_b) {  // for groups of about equal size
  const int avg = std::max(1, max_rows / n_groups);
  return mode == 2 ? choose_plan(dim_a, dim_b, avg, true, 0, n_groups) : choose_plan(avg, dim_b, dim_a, false, 0, n_groups);
}
void dh_gemm_grouped_bf16_tile(int mode, int n_groups, int max_rows, int dim_a, int dim_b, int* rows, int* cols) {
  const GemmPlan p = grouped_plan(mode, n_groups, max_rows, dim_a, dim_b);
  *rows = p.bm;
  *cols = p.bn;
}
int dh_launch_gemm_grouped_bf16(int mode, int n_groups, const int32_t* group_rows, int max_rows, int dim_a, int dim_b,
                                const bf16_t* A, const bf16_t* B, void* C, hipStream_t stream) {
  if (dim_a % 8 || dim_b % 8) DH_FAIL(DH_ERR_SHAPE, "gemm_grouped (bf16): feature dimensions must be multiples of 8 (%d, %d)", dim_a, dim_b);
  if (max_rows == 0) return DH_OK;
  GemmArgs g;
  g.A = A; g.B = B; g.C = C;
  g.bias = nullptr; g.group_rows = group_rows; g.group_mode = mode;
  g.tiles_m = g.tiles_n = g.tiles_per_xcd = 0;
  g.group_part = 0; g.n_groups = n_groups; g.part1_bm = g.part1_bn = 256; g.cus = num_cus(); g.tile_first = 0;
  g.glu_mode = GLU_NONE; g.glu_f = 0; g.glu_in = nullptr; g.glu_out = nullptr; g.ar_blocks = 0;
  GemmPlan p = grouped_plan(mode, n_groups, max_rows, dim_a, dim_b);
  if (mode == 2) { g.M = dim_a; g.N = dim_b; g.K = max_rows; }
  else { g.M = max_rows; g.N = dim_b; g.K = dim_a; }
  g.k_per_split = g.K; g.k_chain = g.n_split = 0;  // no K split
  g.epi = mode == 2 ? EPI_ACC_F32 : EPI_STORE_BF16;
  if (mode == 2) return launch_layout<true, false>(g, p, stream, n_groups);
  if (p.cfg != 0 || n_groups > 64)  // small tiles already, or too many groups for the in-kernel row scan: one launch
    return mode == 0 ? launch_layout<false, false>(g, p, stream, n_groups) : launch_layout<false, true>(g, p, stream, n_groups);
  g.group_part = 1;
  int rc = mode == 0 ? launch_layout<false, false>(g, p, stream, n_groups) : launch_layout<false, true>(g, p, stream, n_groups);
  if (rc != DH_OK) return rc;
  g.group_part = 2;
  g.M = std::min(max_rows, g.part1_bm - 1);  // a remainder is shorter than a large tile
  p.cfg = 1;
  return mode == 0 ? launch_layout<false, false>(g, p, stream, n_groups) : launch_layout<false, true>(g, p, stream, n_groups);
}
