// bf16 causal grouped-query flash attention on the matrix cores, forward and backward.
// Layout: qkv[T, (nq+2nkv)*D] = [q heads | k heads | v heads] (q, k already rotated), o[T, nq*D],
// lse[nq, T] (natural log), delta[nq, T] = rowsum(dO * O).  Tokens are sequence-major; a block
// never crosses a sequence boundary.  D = head_dim is 64 or 128.
// Keys and values are read through AttnGeom: from the packed qkv rows for plain causal attention, or from a
// gathered buffer that also holds the rows of earlier context-parallel ranks (the queries are then the last
// seq - q_off positions of each sequence); dK/dV are written the same way.
//
// All three kernels compute score tiles "transposed" where that keeps per-query statistics
// lane-local: v_mfma_f32_32x32x16_bf16 leaves column j of its result in lane j%32, so
//   forward / dQ : S^T = K Q^T        (column = query  -> running max/sum, lse, delta live in the lane)
//   dK/dV        : S   = Q K^T        (column = key    -> the dK^T, dV^T accumulators keep their column)
// and the probability tile is fed back as the B operand of the next product straight from registers
// (the 8 k-slots of a lane are rows 8*(r/4)+4*(lane/32)+r%4 of two adjacent register quads).  The
// matching A operand (V^T, K^T, dO^T, Q^T: "k" is the token index, the slow dimension in memory)
// comes from LDS through the transposing load ds_read_b64_tr_b16.
//
// 64-token tiles stream global -> LDS directly (see dma.h) through a ring of three slots (two or three in the
// forward kernels, so that two of their blocks fit a compute unit): in the loops in phases the transfer of tile t+2 (t+1) is issued
// right after the barrier that publishes tile t; in the pinned ones (attn_fwd_pinned, attn_bwd_dkv_block at D = 128) the transfers stand between score
// products, tile t+2's beside tile t's (forward: K of t+2 and V of t+1).  A tile is stored
// [token][D] unpadded; the 16-byte chunk c of row r sits at chunk position c ^ swz(r), which makes
// the 16-byte fragment reads (16 consecutive rows, one chunk) and the transposing reads (4
// consecutive rows x 64 bytes) both bank-conflict free for 256-byte rows (D = 128).
// Blocks are launched heaviest first over all heads (the causal work per block grows with its position).
// Long rows of tiles may be cut into chunks whose float32 partial results a small kernel merges in chunk
// order; the chunk length is chosen per launch from a simulation of the launch (pick_chunk below).
// No atomics: dQ is produced per query block, dK/dV per key block, which walks the heads of its group in index order.
#include <algorithm>
#include <map>
#include <mutex>
#include <queue>
#include <tuple>
#include <vector>
#include "common.h"
#include "dma.h"

#define AB_THREADS 256
#define AB_KT 64   // tokens per LDS tile
#define AB_RING 3  // tile slots
// Tile slots of the dQ kernel in a launch of its own: two at D = 128, so that two of its blocks fit a compute unit (64 KiB each,
// 256 registers a lane).  The arithmetic of one block's waves then runs beside the products of the other's: 32 heads x 4096
// tokens 250 -> 205 us, 4 heads x 4096 queries over 12288 keys 167 -> 136 us.  (Two blocks fit anyway at D = 64.)
// The 256 registers are six too few: they go to scratch (28 bytes a lane), most of them around the whole tile loop, the others read
// again on diagonal tiles and for the transfers of a ragged tile only.
// Where rows are cut into chunks, two resident blocks also mean finer chunks (pick_chunk): the float32 partial rows
// then add up over other ranges of keys than with one block a unit, and some results round to the other bf16 neighbour.
__host__ __device__ constexpr int dq_ring(int d) { return d == 128 ? 2 : AB_RING; }

// Work split of the backward kernels.  Along the block's own dimension there are ceil(seq/128) blocks;
// block i has tiles_of(i) tiles to walk and is cut into ceil(tiles/ch) chunks (ch is chosen per launch).  A launch index is
// mapped to (block, chunk) heaviest block first; `pair` numbers the (block, chunk) pairs in natural order.
//
// Positions.  seq = keys per sequence (positions 0..seq-1); the queries of a sequence are its positions
// q_off..seq-1 (q_off = 0: every position; otherwise a multiple of 128, so that query blocks and key blocks
// share one grid of 128-position blocks, of which blocks q_off/128.. hold queries).  Query-side arrays (q in qkv,
// o, dout, lse, delta, dq) are indexed by the local token b*(seq-q_off) + position - q_off; keys, values and
// their gradients by b*seq + position in kv / dkv, rows of ldkv / lddkv elements laid out [k heads | v heads].
struct AttnGeom {
  int seq, q_off, nq, nkv;
  const bf16_t* kv; int ldkv;
  bf16_t* dkv; int lddkv;
  int ch;      // backward kernels: 64-token tiles per chunk
  int nq_all;  // heads * batch (query heads; key/value heads for dK/dV): a launch index is (pair index) * nq_all + (batch * heads + head),
               // so that the heaviest chunks of every head start first
  int grp;     // query heads of a key/value head (dK/dV: a key block walks the tiles of all of them, head after head)
};
struct ChunkMap { int blk, chunk, pair, chunks; };
__host__ __device__ static inline int dq_tiles(int i, int seq) { int e = (i + 1) * 128; return ((e < seq ? e : seq) + AB_KT - 1) / AB_KT; }
__host__ __device__ static inline int dkv_first(int i, int q_off) { return i * 128 > q_off ? i * 128 : q_off; }  // first query position a key block meets
__host__ __device__ static inline int dkv_tiles(int i, int seq, int q_off) { return (seq - dkv_first(i, q_off) + AB_KT - 1) / AB_KT; }
__host__ __device__ static inline int chunks_of(int tiles, int c) { return (tiles + c - 1) / c; }
static int total_pairs_dq(int seq, int q_off, int c) {
  int n = 0;
  for (int i = q_off / 128; i < (seq + 127) / 128; i++) n += chunks_of(dq_tiles(i, seq), c);
  return n;
}
static int total_pairs_dkv(int seq, int q_off, int c, int grp) {
  int n = 0;
  for (int i = 0; i < (seq + 127) / 128; i++) n += chunks_of(grp * dkv_tiles(i, seq, q_off), c);
  return n;
}
// Which of n blocks, of count(v) units each, holds unit id, and how many units lie before that block.  The wave looks at all blocks
// side by side (a count takes an integer division: one after the other they took microseconds).  found == false: id is not among them.
struct UnitOf { int v, rem, before, total; bool found; };
template <class Count>
__device__ __forceinline__ UnitOf find_unit(int id, int n, Count count) {
  const int lane = threadIdx.x & 63, per = (n + 63) >> 6, v0 = lane * per;
  int mine = 0;
  for (int k = 0; k < per; k++) mine += v0 + k < n ? count(v0 + k) : 0;
  int upto = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(upto, d, 64);
    if (lane >= d) upto += t;
  }
  UnitOf u;
  int v = v0, before = upto - mine;
  const bool own = id >= before && id < upto;
  if (own)
    for (int c; id - before >= (c = count(v)); v++) before += c;
  const unsigned long long who = __ballot(own);
  u.found = who != 0;
  u.total = __builtin_amdgcn_readlane(upto, 63);
  const int src = who != 0 ? __builtin_ctzll(who) : 0;
  u.v = __builtin_amdgcn_readlane(v, src);
  u.before = __builtin_amdgcn_readlane(before, src);
  u.rem = id - u.before;
  return u;
}
// Sum of count(k) over first <= k < end, by the whole wave.
template <class Count>
__device__ __forceinline__ int wave_sum(int first, int end, Count count) {
  int s = 0;
  for (int k = first + (int)(threadIdx.x & 63); k < end; k += 64) s += count(k);
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
  return __builtin_amdgcn_readfirstlane(s);
}
// dQ: heaviest = last block; the first block with queries is q_off/128.  (One block after the other: this kernel has no register
// left for find_unit, which doubles what goes to scratch.)
__device__ __forceinline__ ChunkMap map_dq(int id, int seq, int q_off, int total, int c) {
  ChunkMap m;
  int rem = id, after = 0;  // `after` = pairs of the blocks visited before this one
  int i = (seq + 127) / 128 - 1;
  for (;; i--) { int ch = chunks_of(dq_tiles(i, seq), c); if (rem < ch || i == q_off / 128) { m.chunks = ch; break; } rem -= ch; after += ch; }
  m.blk = i; m.chunk = rem; m.pair = total - after - m.chunks + rem;
  return m;
}
// The block with the idx-th longest rest (ties: the earlier block first), found by the whole wave; rest(i) == 0: no unit.
template <class Rest>
__device__ __forceinline__ int nth_rest(int idx, int n, Rest rest) {
  const int lane = threadIdx.x & 63, per = (n + 63) >> 6, v0 = lane * per;
  for (int k = 0; k < per; k++) {
    const int i = v0 + k, mine = i < n ? rest(i) : 0;
    int rank = 0;
    for (int kk = 0; kk < per; kk++) {
      const int other = v0 + kk < n ? rest(v0 + kk) : 0;
      for (int l = 0; l < 64; l++) {
        const int r = __builtin_amdgcn_readlane(other, l);
        rank += r > mine || (r == mine && l * per + kk < i) ? 1 : 0;
      }
    }
    const unsigned long long who = __ballot(mine > 0 && rank == idx);
    if (who != 0) return __builtin_amdgcn_readlane(i, __builtin_ctzll(who));
  }
  return 0;
}
// dK/dV: first every chunk of c tiles (all alike), then what is left of the blocks, longest first: few
// units a compute unit leave a short last round that way only.  In the blocks' order, 8 key/value heads of 4 query heads x 4096
// tokens in chunks of 128 took 502 us: the hardware hands blocks to the shader engines in turn, so the long chunks, each followed by a
// block's short one, met on the same engines.  Unsplit blocks are longest first by themselves.
// Tiles per chunk of a launch that splits no block: more than any block has (a key block has its group's heads x tokens / 64 of them, 2^20 with 64 heads
// and 2^20 tokens).
#define AB_WHOLE (1 << 30)
__device__ __forceinline__ ChunkMap map_dkv(int id, int seq, int q_off, int c, int grp) {
  ChunkMap m;
  if (c >= AB_WHOLE) { m.blk = m.pair = id; m.chunk = 0; m.chunks = 1; return m; }
  const int nblk = (seq + 127) / 128;
  const UnitOf u = find_unit(id, nblk, [&](int i) { return grp * dkv_tiles(i, seq, q_off) / c; });
  m.blk = u.found ? u.v : nth_rest(id - u.total, nblk, [&](int i) { return grp * dkv_tiles(i, seq, q_off) % c; });
  const int tiles = grp * dkv_tiles(m.blk, seq, q_off);
  m.chunk = u.found ? u.rem : tiles / c;
  m.chunks = chunks_of(tiles, c);
  m.pair = wave_sum(0, m.blk, [&](int i) { return chunks_of(grp * dkv_tiles(i, seq, q_off), c); }) + m.chunk;
  return m;
}

typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

#define LOG2E 1.4426950408889634f
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)

// acc += A * B with the accumulator held in the accumulation half of the register file (AGPRs) for the whole
// tile loop: the long-lived gradient accumulators then cost no ordinary registers and no copies.  (This file
// is built with -amdgpu-mfma-vgpr-form, so the short-lived score tiles that the vector ALU post-processes are
// produced in ordinary registers by the intrinsic, with the compiler's own hazard handling.)  The hardware
// interlocks back-to-back accumulation into the same registers; the wait states the compiler would otherwise
// insert around a matrix instruction are written out by hand, since it cannot see into the assembly statement:
// before the instruction (see mfma_acc) and, before anything else reads an accumulator, mfma_acc_settle().
__device__ __forceinline__ void mfma_acc(f32x16& acc, bf16x8 a, bf16x8 b) {
  // two wait states first: an operand fragment may have been written by the vector ALU (the bf16 packing) in the
  // instruction just before, and a matrix instruction must not read such a register that early
  asm("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// acc = 0, produced by the matrix unit so that the accumulator is born in an AGPR; the trailing wait states let
// the result land before any register copy the compiler may place behind this statement.
__device__ __forceinline__ void mfma_acc_zero(f32x16& acc) {
  const bf16x8 z = {0, 0, 0, 0, 0, 0, 0, 0};
  asm volatile("s_nop 3\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %1, 0\n\ts_nop 15\n\ts_nop 15" : "=a"(acc) : "v"(z));
}
__device__ __forceinline__ void mfma_acc_settle(f32x16 (&a)[2]) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(a[0]), "+a"(a[1]));
}
__device__ __forceinline__ void mfma_acc_settle(f32x16 (&a)[4]) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(a[0]), "+a"(a[1]), "+a"(a[2]), "+a"(a[3]));
}
// The same three for loops whose every instruction has its place (attn_fwd_pinned, attn_bwd_dkv_block at D = 128): volatile, so that they stay in the order
// written, and without wait states of their own.  A fragment the vector ALU has written is ready a matrix instruction later, a result two of them later.
__device__ __forceinline__ void mfma_first(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_next(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_grad(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// Wait states between the vector ALU's packing of a fragment and mfma_grad, which has none of its own and hides the hazard from the compiler.  The
// fragment is an operand, so that the packing cannot be scheduled behind them.
__device__ __forceinline__ void frag_settle(bf16x8& f) { asm volatile("s_nop 3" : "+v"(f)); }
// The AGPR placement (AGPR = true) pays where one wave has a SIMD's register file to itself and ordinary registers are short
// (D = 128, one block per compute unit).  With D = 64 everything fits the ordinary registers, and where two waves share the
// file (the dQ kernel at D = 128) they are one budget of 256: there the compiler would only shuttle an AGPR-constrained value
// back and forth (64 moves per tile, dQ 205 -> 250 us at 32 heads x 4096 tokens), so those kernels use the intrinsic.
template <bool AGPR> __device__ __forceinline__ void acc_zero(f32x16& acc) {
  if constexpr (AGPR) mfma_acc_zero(acc);
  else {
#pragma unroll
    for (int r = 0; r < 16; r++) acc[r] = 0.f;
  }
}
template <bool AGPR> __device__ __forceinline__ void acc_mfma(f32x16& acc, bf16x8 a, bf16x8 b) {
  if constexpr (AGPR) mfma_acc(acc, a, b);
  else acc = MFMA(a, b, acc);
}
template <bool AGPR, int N> __device__ __forceinline__ void acc_settle(f32x16 (&a)[N]) {
  if constexpr (AGPR) mfma_acc_settle(a);
}


// Wait states after which the vector ALU may read score tiles.
__device__ __forceinline__ void mfma_settle(f32x16 (&a)[2]) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+v"(a[0]), "+v"(a[1]));
}

template <int D>
struct ATile {
  static constexpr int LD = D;
  static constexpr int ELEMS = AB_KT * D;
  static constexpr int BYTES = ELEMS * 2;
  static constexpr int CPR = D / 8;   // 16-byte chunks per row
  static constexpr int IPW = D / 32;  // transfers per wave per tile (4 waves)
  __device__ static __forceinline__ int swz(int r) { return (((r & 3) << 2) | ((r >> 2) & 3)) & (CPR - 1); }
  // element offset of (row r, column c), c a multiple of 4
  __device__ static __forceinline__ int off(int r, int c) { return r * LD + ((((c >> 3) ^ swz(r)) << 3) | (c & 7)); }
};

// Per-lane byte offsets (relative to the tile's first row in global memory, row stride ld elements)
// of the chunks this wave transfers; rows >= rows_valid are clamped to the last valid row.
template <int D>
__device__ __forceinline__ void tile_voff(uint32_t (&v)[ATile<D>::IPW], int ld, int wave, int lane, int rows_valid) {
  using TL = ATile<D>;
#pragma unroll
  for (int j = 0; j < TL::IPW; j++) {
    const int p = (wave * TL::IPW + j) * 64 + lane;
    const int row = p / TL::CPR, c = (p % TL::CPR) ^ TL::swz(row);
    v[j] = (uint32_t)(((size_t)min(row, rows_valid - 1) * ld + c * 8) * sizeof(bf16_t));
  }
}
template <int D>
__device__ __forceinline__ void tile_dma(const char* base, const uint32_t (&v)[ATile<D>::IPW], uint32_t lds_tile, int wave) {
#pragma unroll
  for (int j = 0; j < ATile<D>::IPW; j++) dma16_base(base, v[j], lds_tile + (wave * ATile<D>::IPW + j) * 1024);
}

// The same with transfer j's KiB as a constant that the hardware adds to both addresses (see dma.h): v[j] is that much less.
template <int D>
__device__ __forceinline__ void tile_dma_at(const char* base, const uint32_t (&v)[ATile<D>::IPW], uint32_t lds_tile, int wave) {
  const uint32_t m = dma_lds(lds_tile + wave * ATile<D>::IPW * 1024);
#pragma unroll
  for (int j = 0; j < ATile<D>::IPW; j++) dma16_at(m, base, v[j], j * 1024);
}

// Byte offsets inside a tile of the two kinds of fragment reads, precomputed per lane.
//   direct: row l32 (+32*mt), columns ks*16 + kg*8 .. +7              -> kdir[ks] (+ mt*32*LD*2)
//   transposed: rows 4*kg + s/4 (+8 for the second read) (+ mt*32 + 16*c), column dt*32 + h16*16 + (s%4)*4
//                                                                      -> tr0[dt], tr1[dt] (+ (mt*32+16c)*LD*2)
// The swizzle of a row only depends on row%16 through bits that the added multiples of 16 (and, for
// the direct reads, 32) leave untouched, so the additions are plain constants.
template <int D>
struct FragAddr {
  int kdir[D / 16], tr0[D / 32], tr1[D / 32];
  __device__ __forceinline__ void init(int lane) {
    using TL = ATile<D>;
    const int l32 = lane & 31, kg = lane >> 5, s16 = lane & 15, h16 = (lane >> 4) & 1;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) kdir[ks] = TL::off(l32, ks * 16 + kg * 8) * 2;
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) {
      tr0[dt] = TL::off(4 * kg + (s16 >> 2), dt * 32 + h16 * 16 + ((s16 & 3) << 2)) * 2;
      tr1[dt] = TL::off(8 + 4 * kg + (s16 >> 2), dt * 32 + h16 * 16 + ((s16 & 3) << 2)) * 2;
    }
  }
};
// Fragment reads take a per-lane pointer (tile base + precomputed lane offset) and a compile-time
// constant byte offset, which the compiler folds into the offset field of the LDS instruction.
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
__device__ __forceinline__ bf16x8 lds_frag(const lds_char* lane_ptr, int const_off) {
  return *reinterpret_cast<const lds_bf16x8*>(lane_ptr + const_off);
}
__device__ __forceinline__ bf16x8 lds_frag_tr(const lds_char* lane_ptr0, const lds_char* lane_ptr1, int const_off) {
  s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lane_ptr0 + const_off));
  s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lane_ptr1 + const_off));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}
// Per-tile lane pointers for one LDS tile.
template <int D>
struct TilePtrs {
  const lds_char* dir[D / 16];
  const lds_char* t0[D / 32];
  const lds_char* t1[D / 32];
  __device__ __forceinline__ void set(const lds_char* tile, const FragAddr<D>& fa) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) dir[ks] = tile + fa.kdir[ks];
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) { t0[dt] = tile + fa.tr0[dt]; t1[dt] = tile + fa.tr1[dt]; }
  }
};
// Registers 8c..8c+7 of a 32x32 result tile as a bf16 B fragment (k-slots = rows 16c+4g+{0..3}, 16c+8+4g+{0..3}).
__device__ __forceinline__ bf16x8 pack_rows(const f32x16& t, int c) {
  bf16x8 f;
#pragma unroll
  for (int i = 0; i < 8; i++) f[i] = (bf16_t)t[8 * c + i];
  return f;
}
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Score tiles of a 64-token LDS tile: acc[mt] = sum over k of T[rows 32 mt .. 32 mt + 31][k] * b[k] (direct fragments
// of the tile behind P against the D-long register fragments b).  A matrix instruction that accumulates into the
// result of the one just before it has to wait for that result, so the products of the two independent tiles are
// issued round robin.  The LDS fragments of the next two k-steps are requested before the products of the current two are
// issued, and the matrix and LDS instructions are pinned in that order (vector arithmetic of the caller may still move
// across), so no product waits for an LDS read issued just before it.
#define SCHED_PIN_MFMA_DS() __builtin_amdgcn_sched_barrier(0x2 | 0x4 | 0x400)  // vector (not matrix), scalar and transcendental arithmetic may cross
template <int D>
__device__ __forceinline__ void score_tiles(f32x16 (&acc)[2], const TilePtrs<D>& P, const bf16x8 (&b)[D / 16]) {
  using TL = ATile<D>;
  constexpr int KS = D / 16;
  const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 fr[2][4];  // two k-steps (two fragments each) per chunk
  auto fetch = [&](int c) {
#pragma unroll
    for (int i = 0; i < 4; i++) fr[c & 1][i] = lds_frag(P.dir[2 * c + (i >> 1)], (i & 1) * 32 * TL::LD * 2);
  };
  fetch(0);
#pragma unroll
  for (int c = 0; c < KS / 2; c++) {
    if (c + 1 < KS / 2) fetch(c + 1);
    SCHED_PIN_MFMA_DS();
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int ks = 2 * c + (i >> 1), mt = i & 1;
      acc[mt] = MFMA(fr[c & 1][i], b[ks], ks == 0 ? z : acc[mt]);
    }
    SCHED_PIN_MFMA_DS();
  }
}
// The backward kernels' two operand pairs, one after the other: S from the tile behind P0 in the first D/16 steps, dP from the
// tile OFF1 bytes further in the next; arith(j) follows the products of dP's step j and turns a part of S into P beside
// them (32 exponentials take about as long as the 16 products of dP).  Fragments are requested AHEAD steps of 64 matrix
// cycles ahead: three where registers allow it, one where a second wave on the SIMD covers the wait.  Every step is pinned
// as written.  dK/dV at 32 heads x 4096 tokens, one wave a SIMD: 335 -> 315 us.
template <int D, int OFF1, int AHEAD, class F>
__device__ __forceinline__ void score_tiles2(f32x16 (&acc0)[2], const TilePtrs<D>& P0, const bf16x8 (&b0)[D / 16],
                                             f32x16 (&acc1)[2], const bf16x8 (&b1)[D / 16], F arith) {
  using TL = ATile<D>;
  constexpr int KS = D / 16;
  const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  bf16x8 fr[AHEAD + 1][2];
  auto fetch = [&](int i) {
#pragma unroll
    for (int mt = 0; mt < 2; mt++) fr[i % (AHEAD + 1)][mt] = lds_frag(P0.dir[i % KS], (i < KS ? 0 : OFF1) + mt * 32 * TL::LD * 2);
  };
#pragma unroll
  for (int i = 0; i < AHEAD; i++) fetch(i);
#pragma unroll
  for (int i = 0; i < 2 * KS; i++) {
    if (i + AHEAD < 2 * KS) fetch(i + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    if (i < KS) {
      acc0[0] = MFMA(fr[i % (AHEAD + 1)][0], b0[i], i == 0 ? z : acc0[0]);
      acc0[1] = MFMA(fr[i % (AHEAD + 1)][1], b0[i], i == 0 ? z : acc0[1]);
    } else {
      acc1[0] = MFMA(fr[i % (AHEAD + 1)][0], b1[i - KS], i == KS ? z : acc1[0]);
      acc1[1] = MFMA(fr[i % (AHEAD + 1)][1], b1[i - KS], i == KS ? z : acc1[1]);
      __builtin_amdgcn_sched_barrier(0);
      arith(i - KS);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// acc[dt] += T[64 x D]^T (transposed fragments of the LDS tile behind P) * src, src = a 64 x 32 score tile held as
// two 32x32 register tiles.  The 64 "k" rows go in four groups of 16 (g = 2*mt + c); the transposed fragments
// of group g+1 are fetched before the products of group g are issued, so no product waits for its own LDS
// read, and between(g) runs after group g's products are issued (independent vector work to overlap them).  The caller has
// fetched group 0 (tr_fetch); NEXT: group 0 of the tile behind P2 is fetched beside the last products.
template <int D> using TrFrags = bf16x8[2][D / 32];
template <int D>
__device__ __forceinline__ void tr_fetch(TrFrags<D>& fr, const TilePtrs<D>& P, int g) {
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) fr[g & 1][dt] = lds_frag_tr(P.t0[dt], P.t1[dt], g * 16 * ATile<D>::LD * 2);
}
template <int D, bool NEXT, bool AGPR, class F>
__device__ __forceinline__ void acc_tile_tr(f32x16 (&acc)[D / 32], TrFrags<D>& fr, const TilePtrs<D>& P, const f32x16 (&src)[2],
                                            const TilePtrs<D>& P2, F between) {
#pragma unroll
  for (int g = 0; g < 4; g++) {
    if (g + 1 < 4) tr_fetch<D>(fr, P, g + 1);
    else if (NEXT) tr_fetch<D>(fr, P2, 0);
    const bf16x8 pf = pack_rows(src[g >> 1], g & 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) acc_mfma<AGPR>(acc[dt], fr[g & 1][dt], pf);
    __builtin_amdgcn_sched_barrier(0);
    between(g);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A row's fragments; zeros for a lane whose row is not `valid` (row: of some row that exists all the same).  Those lanes read a row of zeros: with a branch
// around the loads the compiler copied some of their registers where the two ways met, and a dK/dV block waited for memory twice between its loads (grouped heads, the whole
// backward pass, us: 2 x 264 tokens on 4:1 30.2 -> 29.4, 128 tokens on 8:2 24.1 -> 23.6; forward 4:1 x 4096 36.6 -> 36.2).
__device__ __attribute__((aligned(16))) bf16_t ab_zero_row[128];
template <int D>
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[D / 16], const bf16_t* row, bool valid, int kg) {
  static_assert(D <= 128, "ab_zero_row");
  const bf16_t* src = (valid ? row : ab_zero_row) + kg * 8;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) f[ks] = *reinterpret_cast<const bf16x8*>(src + ks * 16);
}

// Makes the compiler wait here for the global loads that produced the fragments: their first use would
// otherwise be inside the tile loop, and the wait it would place there (a vmcnt count that knows nothing
// of the asynchronous tile transfers) would drain the transfer ring on every step.
template <int N>
__device__ __forceinline__ void pin_frags(const bf16x8 (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; i++) asm volatile("" ::"v"(f[i]));
}
__device__ __forceinline__ void pin_scalar(float v) { asm volatile("" ::"v"(v)); }

// ================================================================================ forward
// Work units of the forward kernel: query block i (128 rows) needs fwd_tiles(i) key tiles; with ch > 0 they
// are cut into chunks of ch tiles (ch even, so that every chunk starts at a tile each of the block's waves
// can see), one launch index per (block, chunk), heaviest block first.  A block with a single chunk writes
// o and lse itself; otherwise every chunk writes its unnormalised float32 output rows with their running
// maximum and sum, and a combine kernel merges the chunks in chunk order.
__host__ __device__ static inline int fwd_tiles(int i, int seq) { int e = (i + 1) * 128; return ((e < seq ? e : seq) + AB_KT - 1) / AB_KT; }
__host__ __device__ static inline int fwd_chunks(int i, int seq, int ch) { return ch > 0 ? (fwd_tiles(i, seq) + ch - 1) / ch : 1; }
static int fwd_units(int seq, int q_off, int ch) {
  int n = 0;
  for (int i = q_off / 128; i < (seq + 127) / 128; i++) n += fwd_chunks(i, seq, ch);
  return n;
}

// Wave w of a block owns query rows i0 + 32w .. +31.  Tile slots: the loop in phases two for K and two for V, so that two blocks share a unit at either head width;
// the pipelined one of D = 128 (attn_fwd_pinned) reads K a tile ahead of V, so a V tile stays a tile longer.
#define AF_RING 2
#define AF_K_RING 2
#define AF_V_RING 3
#define AF_BIAS 4096  // see tile_voff_biased

// A wave's 32 rows x D columns in the transposed accumulator layout (lane l32 = row, kg = lane / 32; quad (dt, q4) of
// a lane is columns dt*32 + 8*q4 + 4*kg .. +3) leave through a wave-private LDS region so that a lane stores 16 bytes
// of a contiguous row segment instead of 16 (float32) or 8 (bf16) bytes scattered over 32 rows.  16-byte chunks are
// XOR-swizzled by row; quad(dt, q4) returns the four values, row_ptr(r) the destination of row r or nullptr.
// The region must not be in use by any wave (block barrier before the first call).
template <int D, typename Quad, typename RowPtr>
__device__ __forceinline__ void wave_rows_out_f32(float* reg, int lane, Quad quad, RowPtr row_ptr) {
  constexpr int NCH = D / 4;  // 16-byte chunks per row
  const int l32 = lane & 31, kg = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const int ch = (dt * 32 + 8 * q4 + 4 * kg) >> 2;
      *reinterpret_cast<f32x4*>(reg + l32 * D + ((ch ^ (l32 & (NCH - 1))) << 2)) = quad(dt, q4);
    }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 32 * NCH / 64; it++) {
    const int row = it * (64 / NCH) + lane / NCH, ch = lane % NCH;
    const f32x4 v = *reinterpret_cast<const f32x4*>(reg + row * D + ((ch ^ (row & (NCH - 1))) << 2));
    float* dst = row_ptr(row);
    if (dst != nullptr) *reinterpret_cast<f32x4*>(dst + ch * 4) = v;
  }
}
template <int D, typename Quad, typename RowPtr>
__device__ __forceinline__ void wave_rows_out_bf16(bf16_t* reg, int lane, Quad quad, RowPtr row_ptr) {
  constexpr int NCH = D / 8;  // 16-byte chunks per row
  const int l32 = lane & 31, kg = lane >> 5;
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const int c0 = dt * 32 + 8 * q4 + 4 * kg;
      const f32x4 v = quad(dt, q4);
      const bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
      *reinterpret_cast<bf16x4*>(reg + l32 * D + ((((c0 >> 3) ^ (l32 & (NCH - 1))) << 3) | (c0 & 4))) = o;
    }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 32 * NCH / 64; it++) {
    const int row = it * (64 / NCH) + lane / NCH, ch = lane % NCH;
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(reg + row * D + ((ch ^ (row & (NCH - 1))) << 3));
    bf16_t* dst = row_ptr(row);
    if (dst != nullptr) *reinterpret_cast<bf16x8*>(dst + ch * 8) = v;
  }
}
#define AF_TAU 8.0f  // log2 of the headroom a row's probabilities may take over its reference maximum
#define AB_PIN() __builtin_amdgcn_sched_barrier(0)

// Both halves of the wave: lane l and lane l ^ 32 get f of the two values.
template <class F>
__device__ __forceinline__ float across_halves(float v, F f) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return f(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}

// Offsets for dma16_at with transfer j's KiB as its constant, which the hardware adds to the LDS and to the memory address; the base is AF_BIAS bytes
// before the tile, so that no offset is negative, whatever the clamped row.
template <int D>
__device__ __forceinline__ void tile_voff_biased(uint32_t (&v)[ATile<D>::IPW], int ld, int wave, int lane, int rows_valid) {
  asm volatile("" : "+v"(lane));  // computed here: shared with the other tiles' offsets it would hold registers through the main loop
  tile_voff<D>(v, ld, wave, lane, rows_valid);
#pragma unroll
  for (int j = 0; j < ATile<D>::IPW; j++) v[j] += AF_BIAS - j * 1024;
}

// The D = 128 tile loop: key tiles [t0, t1) of one unit (q: the wave's rows); a wave stops at its last tile with a visible key, at most one short of t1.
// ot: unnormalised output, m: reference maximum (log2), l: sum of the probabilities.
//
// With the phases one after the other (scores, softmax, P V) a tile took 2190 cycles, about its 1024 of matrix instructions and its 1400 of
// vector ALU added up, although two blocks shared the unit.  Here iteration t forms the scores of tile t+1 beside the exponentials of
// tile t, and the maximum of tile t+1 beside the P V products of tile t; every matrix instruction is volatile and followed by its share of the
// rest, and all of it is pinned.  A barrier an iteration, in its P V half, publishes K(t+2) and V(t+1) and retires K(t+1) and V(t-1), whose slots the
// next iteration fills (tiles behind the unit's end are its last one again, so that every iteration has 8 transfers).
// The same sums in the same order as the loop in phases: the same bits.
//
// Measured alone, both in turn in a loop of launches (us, in phases -> here): 32:8 heads x 4096 tokens 152 -> 141, 8:1 x 8192 175 -> 157, 4:1 x 4096 queries over
// 12288 keys 119 -> 108, 2 x 2048 x 8 heads 43.9 -> 36.7, 16:4 x 1500 32.4 -> 27.8; as one kernel after the other of a layer 32:8 x 4096 160 -> 145, 2 x 2048 x 8
// heads 48 -> 45, 4:1 x 4096 31.4 -> 30.0.  In cycles it is 17 % (290 -> 240 thousand at 32:8 heads; matrix cores busy 41 -> 48 % by counters that also count some 10 us around a
// dispatch): the clock falls from 1.75 to 1.65 GHz, the power limit takes the rest.  Without the LDS reads (results meaningless) the same loop takes 200 thousand cycles and 108 us, so these
// are its largest single cost; two heads of a group a block, which halves them but needs a unit's registers for one block, 149 us there and 135 over 12288 keys,
// 23 instead of 15.7 for 3 x 683 tokens: a block's start and end (6 us, 40 KiB of code to fetch) have nothing beside them.  One block a unit with rings of three and four
// slots: 175.
__device__ __forceinline__ void attn_fwd_pinned(char* smem, const char* kbase, const char* vbase, size_t tstride, int ldkv, int seq, int t0, int t1, int iw,
                                                float scale_log2, const bf16_t* q, f32x16 (&ot)[4], float& m, float& l) {
  constexpr int D = 128, KS = D / 16;
  using TL = ATile<D>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, kg = lane >> 5;
  const int tile_end = min(t1, (iw + 31) / AB_KT + 1), iq = iw + l32;
  const int ragged = seq % AB_KT != 0 ? seq / AB_KT : -1;  // the sequence's last tile if it is not whole
  const lds_char* sm = (const lds_char*)smem;
  const uint32_t ldsKw = lds_address(smem) + wave * (TL::IPW * 1024), ldsVw = ldsKw + AF_K_RING * TL::BYTES;
  auto first_fetch = [&](const char* base, int t, uint32_t lds) {
    t = min(t, t1 - 1);
    uint32_t v[TL::IPW];
    tile_voff_biased<D>(v, ldkv, wave, lane, min(seq - t * AB_KT, AB_KT));
    const uint32_t m0 = dma_lds(lds);
#pragma unroll
    for (int j = 0; j < TL::IPW; j++) dma16_at(m0, base + t * tstride - AF_BIAS, v[j], j * 1024);
  };
  first_fetch(kbase, t0, ldsKw);
  bf16x8 qf[KS];
  load_row_frags<D>(qf, q, iq < seq, kg);
  first_fetch(vbase, t0, ldsVw);
  first_fetch(kbase, t0 + 1, ldsKw + TL::BYTES);
  int kt = min(t0 + 2, t1 - 1), vt = min(t0 + 1, t1 - 1);  // tiles to transfer next
  const char* kp = kbase + kt * tstride - AF_BIAS;
  const char* vp = vbase + vt * tstride - AF_BIAS;
  uint32_t vk[TL::IPW], vv[TL::IPW];
  tile_voff_biased<D>(vk, ldkv, wave, lane, min(seq - kt * AB_KT, AB_KT));
  tile_voff_biased<D>(vv, ldkv, wave, lane, min(seq - vt * AB_KT, AB_KT));

  const lds_char* dir[KS];
  const lds_char* tr0[D / 32];
  const lds_char* tr1[D / 32];
  {
    FragAddr<D> fa;
    fa.init(lane);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) dir[ks] = sm + fa.kdir[ks];
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) {
      tr0[dt] = sm + AF_K_RING * TL::BYTES + fa.tr0[dt];
      tr1[dt] = sm + AF_K_RING * TL::BYTES + fa.tr1[dt];
    }
  }
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) mfma_acc_zero(ot[dt]);
  pin_frags(qf);
#pragma unroll
  for (int ks = 0; ks < KS; ks++) asm volatile("" : "+a"(qf[ks]));
  typedef f32x16 Scores[2];
  bf16x8 fr[4][2];       // K fragments of four k-steps: asked for three steps ahead
  bf16x8 tr[4][D / 32];  // V fragments of the tile's four groups of 16 keys: two groups ahead
  bf16x8 pf[4];          // the groups' packed probabilities
  Scores sa, sb;         // scores, then probabilities, of even and odd iterations
  auto frag = [&](int step, int mt) { fr[step & 3][mt] = lds_frag(dir[step], mt * 32 * TL::LD * 2); };
  auto trfrag = [&](int g, int dt) { tr[g][dt] = lds_frag_tr(tr0[dt], tr1[dt], g * 16 * TL::LD * 2); };
  auto first_frags = [&]() {
#pragma unroll
    for (int step = 0; step < 3; step++) { frag(step, 0); frag(step, 1); }
  };
  auto score = [&](Scores& s, int i) {
    if (i < 2) mfma_first(s[i & 1], fr[0][i & 1], qf[0]);
    else mfma_next(s[i & 1], fr[(i >> 1) & 3][i & 1], qf[i >> 1]);
    if ((i >> 1) + 3 < KS) frag((i >> 1) + 3, i & 1);
  };
  float mx, rs;
  auto prob = [&](Scores& s, int x) {
    float p = fast_exp2(fmaf(s[x >> 4][x & 15], scale_log2, -m));
    rs += p;
    asm volatile("" : "+v"(p), "+v"(rs));  // here, not behind the mask's branch
    s[x >> 4][x & 15] = p;
  };
  auto pack = [&](const Scores& s, int x) {  // elements 2x, 2x+1
    pf[x >> 2][2 * (x & 3)] = (bf16_t)s[x >> 3][2 * (x & 7)];
    pf[x >> 2][2 * (x & 3) + 1] = (bf16_t)s[x >> 3][2 * (x & 7) + 1];
  };
  auto max2 = [&](const Scores& s, int x) {
    const float v = fmaxf(s[x >> 3][2 * (x & 7)], s[x >> 3][2 * (x & 7) + 1]);
    mx = x == 0 ? v : fmaxf(mx, v);
  };
  auto larger = [](float a, float b) { return fmaxf(a, b); };
  auto sum = [](float a, float b) { return a + b; };
  auto mask = [&](Scores& s, int t) {  // the tile crosses the diagonal for this wave: no key above the row
    if (t * AB_KT + AB_KT - 1 <= iw) return;
    mfma_settle(s);
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        s[mt][r] = t * AB_KT + mt * 32 + 8 * (r >> 2) + 4 * kg + (r & 3) > iq ? -INFINITY : s[mt][r];
        if ((r & 3) == 3) AB_PIN();
      }
  };
  int k_slot = 1, v_slot = 0;  // K: the tile whose scores come next, V: the tile whose products come next

  dma_wait<2 * TL::IPW>();
  __syncthreads();  // K(t0)
  first_frags();
#pragma unroll
  for (int i = 0; i < 16; i++) { score(sa, i); AB_PIN(); }
  mfma_settle(sa);
  mask(sa, t0);
#pragma unroll
  for (int x = 0; x < 16; x++) max2(sa, x);
  mx = across_halves(mx, larger);
  m = fmaxf(-INFINITY, mx * scale_log2);  // finite: the unit's first key is visible to every row
  l = 0.f;
  dma_wait<0>();
  __syncthreads();  // V(t0), K(t0+1)
#pragma unroll
  for (int ks = 0; ks < KS; ks++) dir[ks] += TL::BYTES;
  first_frags();

  // The reference maximum m of a row moves only when some row of the wave outgrows its reference by more than
  // 2^AF_TAU (then every row takes its true maximum and the accumulators are rescaled); otherwise the tile's
  // probabilities are formed against the old reference and may reach 2^AF_TAU, which float32 sums and the bf16 P
  // fragments hold without loss of relative precision.  The result depends on m only through rounding: the
  // normalisation by l at the end and lse = m + log2 l use the same reference.  After the first few tiles of a row the
  // rescaling (one multiply per accumulator element per tile) almost never runs.
  auto reference = [&]() {
    const float mnew = mx * scale_log2;
    if (__any(mnew > m + AF_TAU)) {
      mfma_acc_settle(ot);
      const float mn = fmaxf(m, mnew);
      const float alpha = fast_exp2(m - mn);
      l *= alpha;
      m = mn;
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) ot[dt][r] *= alpha;
    }
  };
  // P V of the tile behind tr0: 16 slots, in each `beside(slot)` and its share of the last group's probabilities and of the packing
  auto products = [&](Scores& s, auto beside) {
#pragma unroll
    for (int i = 0; i < 16; i++) {
      mfma_grad(ot[i & 3], tr[i >> 2][i & 3], pf[i >> 2]);
      if (i < 8) trfrag((i >> 2) + 2, i & 3);
      if (i < 4) pack(s, 8 + i);
      if (i < 8) prob(s, 24 + i);
      else if (i < 10) { pack(s, 2 * i - 4); pack(s, 2 * i - 3); }
      beside(i);
      AB_PIN();
    }
  };
  auto step = [&](Scores& s, Scores& next, int t) {
    uint32_t m0 = 0;
    rs = 0.f;
    const int k_next = k_slot ^ 1, v_next = v_slot == AF_V_RING - 1 ? 0 : v_slot + 1;  // these held K(t) and V(t-2)
    // scores of tile t+1 beside three quarters of tile t's probabilities
#pragma unroll
    for (int i = 0; i < 16; i++) {
      score(next, i);
      if (i == 0) m0 = dma_lds(ldsKw + k_next * TL::BYTES);
      if (i == 4) m0 = dma_lds(ldsVw + v_next * TL::BYTES);
      if (i < 4) dma16_at(m0, kp, vk[i], i * 1024);
      else if (i < 8) dma16_at(m0, vp, vv[i - 4], (i - 4) * 1024);
      else trfrag((i - 8) >> 2, i & 3);
#pragma unroll
      for (int x = i * 24 / 16; x < (i + 1) * 24 / 16; x++) prob(s, x);
      if (i >= 6 && i < 10) pack(s, i - 6);
      if (i >= 11 && i < 15) pack(s, i - 7);
      if (i == 15) asm volatile("" : "+v"(pf[0]), "+v"(pf[1]));  // packed by now: the first products, behind this matrix instruction, read them
      AB_PIN();
    }
    mask(next, t + 1);
    // products of tile t beside its last probabilities and the maximum of tile t+1's scores
    products(s, [&](int i) {
      if (i >= 3 && i < 11) { max2(next, 2 * (i - 3)); max2(next, 2 * (i - 3) + 1); }
      if (i >= 4 && i < 8) {
        dir[2 * (i - 4)] += (k_next - k_slot) * TL::BYTES;
        dir[2 * (i - 4) + 1] += (k_next - k_slot) * TL::BYTES;
      }
      if (i == 9) l += across_halves(rs, sum);
      if (i == 11) {
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        mx = across_halves(mx, larger);
      }
      if (i >= 12 && i < 15) { frag(i - 12, 0); frag(i - 12, 1); }
      if (i >= 12) {
        tr0[i & 3] += (v_next - v_slot) * TL::BYTES;
        tr1[i & 3] += (v_next - v_slot) * TL::BYTES;
      }
    });
    k_slot = k_next;
    v_slot = v_next;
    if (kt < t1 - 1) {
      kp += tstride;
      if (++kt == ragged) tile_voff_biased<D>(vk, ldkv, wave, lane, seq - kt * AB_KT);
    }
    if (vt < t1 - 1) {
      vp += tstride;
      if (++vt == ragged) tile_voff_biased<D>(vv, ldkv, wave, lane, seq - vt * AB_KT);
    }
    reference();
  };
  int t = t0;
  for (; t + 2 < tile_end; t += 2) {
    step(sa, sb, t);
    step(sb, sa, t + 1);
  }
  if (t + 1 < tile_end) {
    step(sa, sb, t);
    sa[0] = sb[0];
    sa[1] = sb[1];
  }
  // the wave's last tile
  if (tile_end < t1) {  // other waves go on: this wave's share of their last V tile
    const uint32_t m0 = dma_lds(ldsVw + (v_slot == AF_V_RING - 1 ? 0 : v_slot + 1) * TL::BYTES);
#pragma unroll
    for (int j = 0; j < TL::IPW; j++) dma16_at(m0, vp, vv[j], j * 1024);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  }
#pragma unroll
  for (int i = 0; i < 8; i++) trfrag(i >> 2, i & 3);
  rs = 0.f;
#pragma unroll
  for (int x = 0; x < 24; x++) prob(sa, x);
#pragma unroll
  for (int x = 0; x < 8; x++) pack(sa, x);
  AB_PIN();
  frag_settle(pf[1]);
  frag_settle(pf[0]);
  products(sa, [](int) {});
  l += across_halves(rs, sum);
  mfma_acc_settle(ot);
  dma_wait<0>();  // the rings' memory is used again
}

// Positions of a unit's rows, common to the kernels below.
struct FwdUnit { int blk, chunk, nchunks, pair; };
__device__ __forceinline__ FwdUnit fwd_unit(int launch, int seq, int qb0, int ch, int units) {
  FwdUnit f = {0, 0, 1, 0};
  if (ch == 0) {
    f.pair = units - 1 - launch;
    f.blk = qb0 + f.pair;
  } else {  // heaviest block first; `pair` numbers the (block, chunk) units in natural order
    const int last = (seq + 127) / 128 - 1;
    const UnitOf u = find_unit(launch, last - qb0 + 1, [&](int v) { return fwd_chunks(last - v, seq, ch); });
    f.blk = last - u.v;
    f.nchunks = fwd_chunks(f.blk, seq, ch);
    f.chunk = u.rem;
    f.pair = units - u.before - f.nchunks + u.rem;
  }
  return f;
}
// A wave's 32 rows leave: the unit's partial result, or the final rows and lse.  unit: index of the partial result.
template <int D>
__device__ __forceinline__ void fwd_rows_out(char* smem, const FwdUnit& u, size_t unit, int seq, int iw, int lane, int wave, const f32x16 (&ot)[D / 32], float m,
                                             float l, bf16_t* orow, size_t ldo, float* lse_row, float* part_o, float* part_ml) {
  const int l32 = lane & 31, iq = iw + l32, r0 = wave * 32;
  if (u.nchunks > 1) {  // partial result of this chunk
    wave_rows_out_f32<D>(
        reinterpret_cast<float*>(smem) + wave * (32 * D), lane,
        [&](int dt, int q4) { return f32x4{ot[dt][4 * q4], ot[dt][4 * q4 + 1], ot[dt][4 * q4 + 2], ot[dt][4 * q4 + 3]}; },
        [&](int r) { return iw + r < seq ? part_o + (unit * 128 + r0 + r) * D : nullptr; });
    if (iq < seq && lane < 32) {
      part_ml[(unit * 128 + r0 + l32) * 2] = m;
      part_ml[(unit * 128 + r0 + l32) * 2 + 1] = l;
    }
    return;
  }
  const float inv = 1.0f / l;
  wave_rows_out_bf16<D>(
      reinterpret_cast<bf16_t*>(smem) + wave * (32 * D), lane,
      [&](int dt, int q4) {
        return f32x4{ot[dt][4 * q4] * inv, ot[dt][4 * q4 + 1] * inv, ot[dt][4 * q4 + 2] * inv, ot[dt][4 * q4 + 3] * inv};
      },
      [&](int r) { return iw + r < seq ? orow + (size_t)r * ldo : nullptr; });
  if (iq < seq && lane < 32) lse_row[l32] = (m + log2f(l)) * 0.6931471805599453f;
}

// grid (units * nq * batch), D = 128
__global__ __launch_bounds__(AB_THREADS, 2) void attn_fwd_pinned_bf16_kernel(const AttnGeom g, const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                                             float* __restrict__ lse, int T, float scale_log2, int ch, int units,
                                                                             float* __restrict__ part_o, float* __restrict__ part_ml) {
  constexpr int D = 128;
  extern __shared__ __attribute__((aligned(1024))) char smem[];  // K ring, then V ring
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int seq = g.seq, nq = g.nq, nkv = g.nkv, ldkv = g.ldkv, ld = (nq + 2 * nkv) * D;
  const int hb = blockIdx.x % g.nq_all, h = hb % nq, b = hb / nq, hk = h / (nq / nkv);
  const FwdUnit u = fwd_unit(blockIdx.x / g.nq_all, seq, g.q_off / 128, ch, units);
  const int i0 = u.blk * 128, iw = i0 + wave * 32;  // positions in the sequence
  const size_t ktok0 = (size_t)b * seq;
  const long long qtok0 = (long long)b * (seq - g.q_off) - g.q_off;  // local token of position p = qtok0 + p
  const char* kbase = reinterpret_cast<const char*>(g.kv + ktok0 * ldkv + (size_t)hk * D);
  const char* vbase = reinterpret_cast<const char*>(g.kv + ktok0 * ldkv + (size_t)(nkv + hk) * D);
  const int tiles_all = (min(seq, i0 + 128) + AB_KT - 1) / AB_KT;  // keys needed by this block: [0, 64*tiles_all)
  const int t0 = u.chunk * ch, t1 = ch == 0 ? tiles_all : min(tiles_all, t0 + ch);  // this unit: tiles [t0, t1)
  f32x16 ot[D / 32];
  float m, l;
  attn_fwd_pinned(smem, kbase, vbase, (size_t)AB_KT * ldkv * sizeof(bf16_t), ldkv, seq, t0, t1, iw, scale_log2,
                  qkv + (size_t)(qtok0 + min(iw + (lane & 31), seq - 1)) * ld + (size_t)h * D, ot, m, l);
  __syncthreads();  // every wave is done with the K/V rings: their LDS serves the output turn
  fwd_rows_out<D>(smem, u, ((size_t)b * nq + h) * units + u.pair, seq, iw, lane, wave, ot, m, l, o + (size_t)(qtok0 + iw) * nq * D + (size_t)h * D,
                  (size_t)nq * D, lse + (size_t)h * T + qtok0 + iw, part_o, part_ml);
}

// The loop in phases: D = 64, and units too short for a pipeline.  grid (units * nq * batch)
template <int D>
__global__ __launch_bounds__(AB_THREADS, 2) void attn_fwd_bf16_kernel(const AttnGeom g, const bf16_t* __restrict__ qkv,
                                                                   bf16_t* __restrict__ o, float* __restrict__ lse, int T,
                                                                   float scale_log2, int ch, int units,
                                                                   float* __restrict__ part_o, float* __restrict__ part_ml) {
  using TL = ATile<D>;
  extern __shared__ __attribute__((aligned(1024))) char smem[];  // K ring, then V ring
  const lds_char* sm = (const lds_char*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, kg = lane >> 5;
  const int seq = g.seq, nq = g.nq, nkv = g.nkv, ldkv = g.ldkv;
  const int hb = blockIdx.x % g.nq_all;
  const int h = hb % nq, b = hb / nq, hk = h / (nq / nkv);
  const int ld = (nq + 2 * nkv) * D;
  const FwdUnit u = fwd_unit(blockIdx.x / g.nq_all, seq, g.q_off / 128, ch, units);
  const int i0 = u.blk * 128, iw = i0 + wave * 32, iq = iw + l32;  // positions in the sequence
  const size_t ktok0 = (size_t)b * seq;
  const long long qtok0 = (long long)b * (seq - g.q_off) - g.q_off;  // local token of position p = qtok0 + p
  const char* kbase = reinterpret_cast<const char*>(g.kv + ktok0 * ldkv + (size_t)hk * D);
  const char* vbase = reinterpret_cast<const char*>(g.kv + ktok0 * ldkv + (size_t)(nkv + hk) * D);
  const size_t tstride = (size_t)AB_KT * ldkv * sizeof(bf16_t);

  bf16x8 qf[D / 16];
  load_row_frags<D>(qf, qkv + (size_t)(qtok0 + min(iq, seq - 1)) * ld + (size_t)h * D, iq < seq, kg);
  f32x16 ot[D / 32];
  float m = -INFINITY, l = 0.f;
  const int tiles_all = (min(seq, i0 + 128) + AB_KT - 1) / AB_KT;  // keys needed by this block: [0, 64*tiles_all)
  const int t_begin = u.chunk * ch, ntiles = ch == 0 ? tiles_all : min(tiles_all, t_begin + ch);  // this unit: [t_begin, ntiles)
  pin_frags(qf);
  FragAddr<D> fa;
  fa.init(lane);
  uint32_t voff[TL::IPW];
  tile_voff<D>(voff, ldkv, wave, lane, AB_KT);
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) ot[dt][r] = 0.f;
  const uint32_t ldsK = lds_address(smem), ldsV = ldsK + AF_RING * TL::BYTES;
  auto issue = [&](int t) {
    const int slot = (t - t_begin) % AF_RING, valid = seq - t * AB_KT;
    if (valid >= AB_KT) {
      tile_dma<D>(kbase + t * tstride, voff, ldsK + slot * TL::BYTES, wave);
      tile_dma<D>(vbase + t * tstride, voff, ldsV + slot * TL::BYTES, wave);
    } else {
      uint32_t vc[TL::IPW];
      tile_voff<D>(vc, ldkv, wave, lane, valid);
      tile_dma<D>(kbase + t * tstride, vc, ldsK + slot * TL::BYTES, wave);
      tile_dma<D>(vbase + t * tstride, vc, ldsV + slot * TL::BYTES, wave);
    }
  };
  issue(t_begin);
  int slot = 0;
  for (int t = t_begin; t < ntiles; t++, slot ^= 1) {
    dma_wait<0>();
    __syncthreads();  // tile t is visible; every wave is done with tile t-1, whose slot tile t+1 reuses
    if (t + 1 < ntiles) issue(t + 1);
    const int kb = t * AB_KT;
    if (kb > iw + 31) continue;  // no key of the tile is visible to any row of this wave
    TilePtrs<D> Kp, Vp;
    Kp.set(sm + slot * TL::BYTES, fa);
    Vp.set(sm + (AF_RING + slot) * TL::BYTES, fa);
    f32x16 st[2];
    score_tiles<D>(st, Kp, qf);
    if (kb + AB_KT - 1 > iw) {  // the tile crosses the diagonal for this wave: mask keys above the row
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int r = 0; r < 16; r++)
          if (kb + mt * 32 + 8 * (r >> 2) + 4 * kg + (r & 3) > iq) st[mt][r] = -INFINITY;
    }
    float mx = fmaxf(st[0][0], st[1][0]);
#pragma unroll
    for (int r = 1; r < 16; r++) mx = fmaxf(mx, fmaxf(st[0][r], st[1][r]));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // The reference maximum moves as in attn_fwd_pinned.
    const float mnew = mx * scale_log2;  // finite from the unit's first tile on: its first key is visible to every row
    float rs = 0.f;
    if (__any(mnew > m + AF_TAU)) {
      const float mn = fmaxf(m, mnew);
      const float alpha = fast_exp2(m - mn);
      l *= alpha;
      m = mn;
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
        for (int r = 0; r < 16; r++) ot[dt][r] *= alpha;
    }
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const float p = fast_exp2(fmaf(st[mt][r], scale_log2, -m));
        st[mt][r] = p;
        rs += p;
      }
    rs += __shfl_xor(rs, 32, 64);
    l += rs;
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
      for (int c = 0; c < 2; c++) {
        const bf16x8 pf = pack_rows(st[mt], c);
        const int ro = (mt * 32 + 16 * c) * TL::LD * 2;
#pragma unroll
        for (int dt = 0; dt < D / 32; dt++) ot[dt] = MFMA(lds_frag_tr(Vp.t0[dt], Vp.t1[dt], ro), pf, ot[dt]);
      }
  }
  __syncthreads();  // every wave is done with the K/V rings: their LDS serves the output turn
  fwd_rows_out<D>(smem, u, ((size_t)b * nq + h) * units + u.pair, seq, iw, lane, wave, ot, m, l, o + (size_t)(qtok0 + iw) * nq * D + (size_t)h * D,
                  (size_t)nq * D, lse + (size_t)h * T + qtok0 + iw, part_o, part_ml);
}

// Merges the chunks of the query blocks that were split: with M = max_c m_c, o = sum_c 2^(m_c-M) o_c / L,
// L = sum_c 2^(m_c-M) l_c, lse = (M + log2 L) ln 2; chunks are added in chunk order.
// grid (8 * blocks, nq, batch): a 256-thread block merges 16 rows, a thread D/16 columns of one row.
template <int D>
__global__ __launch_bounds__(256) void attn_fwd_combine_kernel(int seq, int q_off, int nq, int ch, int units, const float* __restrict__ part_o,
                                                               const float* __restrict__ part_ml, bf16_t* __restrict__ o,
                                                               float* __restrict__ lse, int T) {
  const int blk = q_off / 128 + (blockIdx.x >> 3), h = blockIdx.y, b = blockIdx.z;
  const int nchunks = fwd_chunks(blk, seq, ch);
  if (nchunks == 1) return;
  const int r = (blockIdx.x & 7) * 16 + (threadIdx.x >> 4), pos = blk * 128 + r;
  const int pair0 = wave_sum(q_off / 128, blk, [&](int i) { return fwd_chunks(i, seq, ch); });
  if (pos >= seq) return;
  const size_t unit0 = ((size_t)b * nq + h) * units + pair0;
  constexpr int CPT = D / 16;  // columns per thread
  const int c0 = (threadIdx.x & 15) * CPT;
  const float* ml = part_ml + (unit0 * 128 + r) * 2;
  float M = -INFINITY;
  for (int c = 0; c < nchunks; c++) M = fmaxf(M, ml[(size_t)c * 256]);
  float L = 0.f, acc[CPT];
#pragma unroll
  for (int i = 0; i < CPT; i++) acc[i] = 0.f;
  for (int c = 0; c < nchunks; c++) {
    const float w = exp2f(ml[(size_t)c * 256] - M);
    L += w * ml[(size_t)c * 256 + 1];
    const float* po = part_o + ((unit0 + c) * 128 + r) * D + c0;
#pragma unroll
    for (int i = 0; i < CPT; i += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(po + i);
      acc[i] += w * v[0]; acc[i + 1] += w * v[1]; acc[i + 2] += w * v[2]; acc[i + 3] += w * v[3];
    }
  }
  const float inv = 1.0f / L;
  const size_t tok = (size_t)b * (seq - q_off) + (pos - q_off);
  bf16_t* orow = o + tok * (size_t)nq * D + (size_t)h * D + c0;
#pragma unroll
  for (int i = 0; i < CPT; i += 4) {
    bf16x4 v = {(bf16_t)(acc[i] * inv), (bf16_t)(acc[i + 1] * inv), (bf16_t)(acc[i + 2] * inv), (bf16_t)(acc[i + 3] * inv)};
    *reinterpret_cast<bf16x4*>(orow + i) = v;
  }
  if (c0 == 0) lse[(size_t)h * T + tok] = (M + log2f(L)) * 0.6931471805599453f;
}

// ================================================================================ backward: dQ
// Same tiling as the forward kernel.  dQ^T = sum over key tiles of K^T dS^T, dS^T = P^T (dP^T - delta),
// P^T = exp2(S^T*scale_log2 - lse2), dP^T = V dO^T.
// Every block forms the per-row statistics delta[h,t] = sum_c dO[t,h,c] O[t,h,c] and lse2[h,t] = lse[h,t] log2(e) of its
// own rows itself (a row's two lanes each hold half of dO).  The dK/dV blocks read them from memory: when the dQ blocks
// are launched ahead of them, the block of a query block's first chunk stores them (delta_out != nullptr); when both
// kinds share one launch, attn_bwd_prep_kernel has filled the arrays.
template <int D, int RING>
__device__ __forceinline__ void attn_bwd_dq_block(const int bid, const AttnGeom& g, const bf16_t* __restrict__ qkv,
                                                  const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                                                  const float* __restrict__ lse, float* __restrict__ lse2_out,
                                                  float* __restrict__ delta_out, bf16_t* __restrict__ dqkv,
                                                  float* __restrict__ part, int pairs, int T, float scale, float scale_log2) {
  using TL = ATile<D>;
  constexpr bool AGPR = D == 128 && RING > 2;
  extern __shared__ __attribute__((aligned(1024))) char smem[];  // K ring, then V ring
  const lds_char* sm = (const lds_char*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, kg = lane >> 5;
  const int seq = g.seq, nq = g.nq, nkv = g.nkv, ldkv = g.ldkv;
  const int hb = bid % g.nq_all;
  const int h = hb % nq, b = hb / nq, hk = h / (nq / nkv);
  const int ld = (nq + 2 * nkv) * D;
  const ChunkMap cm = map_dq(bid / g.nq_all, seq, g.q_off, pairs, g.ch);
  const int i0 = cm.blk * 128, iw = i0 + wave * 32, iq = iw + l32;
  const size_t ktok0 = (size_t)b * seq;
  const long long qtok0 = (long long)b * (seq - g.q_off) - g.q_off;  // local token of position p = qtok0 + p
  const char* kbase = reinterpret_cast<const char*>(g.kv + ktok0 * ldkv + (size_t)hk * D);
  const char* vbase = reinterpret_cast<const char*>(g.kv + ktok0 * ldkv + (size_t)(nkv + hk) * D);
  const size_t tstride = (size_t)AB_KT * ldkv * sizeof(bf16_t);

  bf16x8 qf[D / 16], dof[D / 16];
  const size_t qrow = (size_t)(qtok0 + min(iq, seq - 1));
  load_row_frags<D>(qf, qkv + qrow * ld + (size_t)h * D, iq < seq, kg);
  load_row_frags<D>(dof, dout + qrow * (size_t)nq * D + (size_t)h * D, iq < seq, kg);
  const float l2 = lse[(size_t)h * T + qrow] * LOG2E;
  float dl = 0.f;
  {
    bf16x8 of[D / 16];
    load_row_frags<D>(of, o + qrow * (size_t)nq * D + (size_t)h * D, iq < seq, kg);
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++)
#pragma unroll
      for (int e = 0; e < 8; e++) dl = fmaf((float)dof[ks][e], (float)of[ks][e], dl);
    dl += __shfl_xor(dl, 32, 64);  // the row's other half (the same number attn_bwd_prep_kernel stores for the dK/dV blocks)
    if (delta_out != nullptr && cm.chunk == 0 && kg == 0 && iq < seq) {  // launched ahead of the dK/dV kernel: store them for it
      delta_out[(size_t)h * T + qrow] = dl;
      lse2_out[(size_t)h * T + qrow] = l2;
    }
  }
  f32x16 dqt[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) acc_zero<AGPR>(dqt[dt]);

  FragAddr<D> fa;
  fa.init(lane);
  uint32_t voff[TL::IPW];
  tile_voff<D>(voff, ldkv, wave, lane, AB_KT);
  const uint32_t ldsK = lds_address(smem), ldsV = ldsK + RING * TL::BYTES;
  const int t0 = cm.chunk * g.ch, ntiles = min(dq_tiles(cm.blk, seq), t0 + g.ch);  // this block walks key tiles [t0, ntiles)
  auto issue = [&](int t, int slot) {
    const int valid = seq - t * AB_KT;
    if (valid >= AB_KT) {
      tile_dma<D>(kbase + t * tstride, voff, ldsK + slot * TL::BYTES, wave);
      tile_dma<D>(vbase + t * tstride, voff, ldsV + slot * TL::BYTES, wave);
    } else {
      uint32_t vc[TL::IPW];
      tile_voff<D>(vc, ldkv, wave, lane, valid);
      tile_dma<D>(kbase + t * tstride, vc, ldsK + slot * TL::BYTES, wave);
      tile_dma<D>(vbase + t * tstride, vc, ldsV + slot * TL::BYTES, wave);
    }
  };
  pin_frags(qf);
  pin_frags(dof);
  pin_scalar(l2);
  pin_scalar(dl);
  issue(t0, 0);
  if (RING > 2 && t0 + 1 < ntiles) issue(t0 + 1, 1);
  int slot = 0;
  for (int t = t0; t < ntiles; t++, slot = slot == RING - 1 ? 0 : slot + 1) {
    if (RING > 2 && t + 1 < ntiles) dma_wait<2 * TL::IPW>(); else dma_wait<0>();
    __syncthreads();  // tile t is visible; every wave is done with tile t-1, whose slot is filled next
    if (t + RING - 1 < ntiles) issue(t + RING - 1, slot == 0 ? RING - 1 : slot - 1);
    const int kb = t * AB_KT;
    if (kb > iw + 31) continue;
    TilePtrs<D> Kp;
    Kp.set(sm + slot * TL::BYTES, fa);
    f32x16 st[2], dp[2];
    // P^T from S^T beside the dP^T products
    score_tiles2<D, RING * TL::BYTES, (RING == 2 ? 1 : 3)>(st, Kp, qf, dp, dof, [&](int j) {
      constexpr int N = 32 / (D / 16);
#pragma unroll
      for (int i = 0; i < N; i++) {
        const int x = j * N + i;
        st[x >> 4][x & 15] = fast_exp2(fmaf(st[x >> 4][x & 15], scale_log2, -l2));
      }
    });
    TrFrags<D> fr;
    tr_fetch<D>(fr, Kp, 0);
    if (kb + AB_KT - 1 > iw) {
#pragma unroll
      for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int r = 0; r < 16; r++)
          if (kb + mt * 32 + 8 * (r >> 2) + 4 * kg + (r & 3) > iq) st[mt][r] = 0.f;
    }
    // dS^T = P^T (dP^T - delta), one quarter (8 registers of a tile) ahead of the products that consume it
    auto ds_quarter = [&](int g) {
#pragma unroll
      for (int r = 0; r < 8; r++) st[g >> 1][8 * (g & 1) + r] *= dp[g >> 1][8 * (g & 1) + r] - dl;
    };
    ds_quarter(0);
    acc_tile_tr<D, false, AGPR>(dqt, fr, Kp, st, Kp, [&](int g) { if (g + 1 < 4) ds_quarter(g + 1); });
  }
  acc_settle<AGPR>(dqt);
  __syncthreads();  // every wave is done with the K/V rings: their LDS serves the output turn
  if (cm.chunks > 1) {  // float32 partial of this chunk: part[batch][head][pair][128 rows][D], unscaled
    float* rows = part + ((((size_t)b * nq + h) * pairs + cm.pair) * 128 + wave * 32) * D;
    wave_rows_out_f32<D>(
        reinterpret_cast<float*>(smem) + wave * (32 * D), lane,
        [&](int dt, int q4) { return f32x4{dqt[dt][4 * q4], dqt[dt][4 * q4 + 1], dqt[dt][4 * q4 + 2], dqt[dt][4 * q4 + 3]}; },
        [&](int r) { return rows + (size_t)r * D; });
  } else {
    wave_rows_out_bf16<D>(
        reinterpret_cast<bf16_t*>(smem) + wave * (32 * D), lane,
        [&](int dt, int q4) {
          return f32x4{dqt[dt][4 * q4] * scale, dqt[dt][4 * q4 + 1] * scale, dqt[dt][4 * q4 + 2] * scale, dqt[dt][4 * q4 + 3] * scale};
        },
        [&](int r) { return iw + r < seq ? dqkv + (size_t)(qtok0 + iw + r) * ld + (size_t)h * D : nullptr; });
  }
}

// dq[token][head] = scale * sum over the chunks of the token's query block (ascending) of the partials.
// grid (16*query blocks, nq, batch), 256 threads: a block owns 8 rows of a query block, thread = (row, 4 columns).
template <int D>
__device__ __forceinline__ void attn_bwd_dq_reduce_block(int bx, int by, int bz, const float* __restrict__ part,
                                                         bf16_t* __restrict__ dqkv, int seq, int q_off, int nq, int nkv, int pairs,
                                                         int cl, float scale) {
  const int i = q_off / 128 + (bx >> 4), r0 = (bx & 15) * 8, h = by, b = bz, ld = (nq + 2 * nkv) * D;
  const int ch = chunks_of(dq_tiles(i, seq), cl);
  if (ch == 1) return;  // written by its only chunk
  const int base = wave_sum(q_off / 128, i, [&](int k) { return chunks_of(dq_tiles(k, seq), cl); });
  const float* p0 = part + (((size_t)b * nq + h) * pairs + base) * 128 * D;
  for (int e = threadIdx.x; e < 8 * D / 4; e += 256) {
    const int row = r0 + e / (D / 4), c4 = (e % (D / 4)) * 4;
    if (i * 128 + row >= seq) continue;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < ch; c++) s += __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p0 + ((size_t)c * 128 + row) * D + c4));
    bf16x4 o = {(bf16_t)(s[0] * scale), (bf16_t)(s[1] * scale), (bf16_t)(s[2] * scale), (bf16_t)(s[3] * scale)};
    *reinterpret_cast<bf16x4*>(dqkv + ((size_t)b * (seq - q_off) + (i * 128 + row - q_off)) * ld + (size_t)h * D + c4) = o;
  }
}

// ================================================================================ backward: dK, dV
// grid (pairs * nkv * batch): one block per (key block, chunk, key/value head); wave w owns keys
// j0 + 32w .. +31 and keeps their K, V fragments and the dK^T, dV^T accumulators in registers while
// 64-query tiles of Q and dO stream through LDS: those of the group's first query head, then those of the next, and so on
// (the keys are the same), cut into chunks of g.ch tiles wherever that falls.  A key block of one chunk writes dK, dV; the
// chunks of the others write float32 partials part[batch][kv head][pair][128 keys][dK | dV] that
// attn_bwd_reduce_kernel (its dK/dV part) adds in chunk order.  Against a block per query head, whose partials of every head went
// through memory, the whole backward pass (us, chunk lengths as they were): 4:1 heads x 4096 tokens 103 -> 93, 4096 queries over 12288 keys 371 -> 315,
// 32:8 x 4096 508 -> 471, 16:4 x 1500 86 -> 81, 8:1 x 8192 499 -> 493; D = 64, 4:1 x 8192 210 -> 164, 16:4 x 3010 135 -> 115, 16:2 x 5000 234 -> 229.
template <int D>
__device__ __forceinline__ void attn_bwd_dkv_block(const int bid, const AttnGeom& g, const bf16_t* __restrict__ qkv,
                                                   const bf16_t* __restrict__ dout, const float* __restrict__ lse2,
                                                   const float* __restrict__ delta, float* __restrict__ part, int pairs, int T,
                                                   float scale, float scale_log2) {
  using TL = ATile<D>;
  constexpr bool AGPR = D == 128;
  extern __shared__ __attribute__((aligned(1024))) char smem[];  // Q ring, dO ring, lse2 ring, delta ring
  const lds_char* sm = (const lds_char*)smem;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, kg = lane >> 5;
  const int seq = g.seq, nq = g.nq, nkv = g.nkv;
  const int hb = bid % g.nq_all;
  const int hk = hb % nkv, b = hb / nkv, hq = hk * g.grp;  // hq: the group's first query head
  const int ld = (nq + 2 * nkv) * D, ldo = nq * D;
  const ChunkMap cm = map_dkv(bid / g.nq_all, seq, g.q_off, g.ch, g.grp);
  const int j0 = cm.blk * 128, jw = j0 + wave * 32, jk = jw + l32;  // key positions in the sequence (block 0 is the heaviest)
  const int q0 = dkv_first(cm.blk, g.q_off);                        // first query position this key block meets
  const size_t ktok0 = (size_t)b * seq;
  const size_t qtok = (size_t)b * (seq - g.q_off) + (q0 - g.q_off);  // local token of position q0
  const char* qbase = reinterpret_cast<const char*>(qkv + qtok * ld + (size_t)hq * D);
  const char* obase = reinterpret_cast<const char*>(dout + qtok * ldo + (size_t)hq * D);
  const float* lrow = lse2 + (size_t)hq * T + qtok;
  const float* drow = delta + (size_t)hq * T + qtok;
  float* lse_s = reinterpret_cast<float*>(smem + 2 * AB_RING * TL::BYTES);
  float* del_s = lse_s + AB_RING * AB_KT;

  bf16x8 kf[D / 16], vf[D / 16];
  const int jkc = min(jk, seq - 1);
  load_row_frags<D>(kf, g.kv + (ktok0 + jkc) * g.ldkv + (size_t)hk * D, jk < seq, kg);
  load_row_frags<D>(vf, g.kv + (ktok0 + jkc) * g.ldkv + (size_t)(nkv + hk) * D, jk < seq, kg);
  f32x16 dkt[D / 32], dvt[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) { acc_zero<AGPR>(dkt[dt]); acc_zero<AGPR>(dvt[dt]); }

  FragAddr<D> fa;
  fa.init(lane);
  uint32_t vq[TL::IPW], vo[TL::IPW];
  tile_voff<D>(vq, ld, wave, lane, AB_KT);
  tile_voff<D>(vo, ldo, wave, lane, AB_KT);
#pragma unroll
  for (int j = 0; j < TL::IPW; j++) { vq[j] -= j * 1024; vo[j] -= j * 1024; }  // for tile_dma_at: transfer j moves rows from 512 j / D on, of at least 2 D bytes
  const uint32_t ldsQ = lds_address(smem), ldsO = ldsQ + AB_RING * TL::BYTES;
  // The block's tiles: nt query tiles q0 + 64*t of each head of the group, counted through; this chunk walks [f0, f1).
  const int nt = dkv_tiles(cm.blk, seq, g.q_off), f0 = cm.chunk * g.ch, f1 = min(g.grp * nt, f0 + g.ch);
  const size_t qstride = (size_t)AB_KT * ld * sizeof(bf16_t), ostride = (size_t)AB_KT * ldo * sizeof(bf16_t);
  int gi = f0 / nt, ti = f0 - gi * nt;  // head of the group and tile to transfer next
  int tc = ti;                          // tile to work off next
  // per-row statistics of a tile (64 floats each): even waves transfer lse2, odd waves delta (waves 2 and 3
  // repeat what waves 0 and 1 transfer, which keeps the transfer count of all waves equal)
  const uint32_t ldsS = ldsQ + 2 * AB_RING * TL::BYTES + (wave & 1) * AB_RING * AB_KT * sizeof(float);
  const float* srow = (wave & 1) ? drow : lrow;
  pin_frags(kf);
  pin_frags(vf);
  auto issue = [&](int slot) {
    const int row0 = q0 + ti * AB_KT, valid = seq - row0;
    const char* qp = qbase + ti * qstride + gi * (D * sizeof(bf16_t));
    const char* op = obase + ti * ostride + gi * (D * sizeof(bf16_t));
    if (valid >= AB_KT) {
      tile_dma_at<D>(qp, vq, ldsQ + slot * TL::BYTES, wave);
      tile_dma_at<D>(op, vo, ldsO + slot * TL::BYTES, wave);
    } else {
      uint32_t vc[TL::IPW];
      tile_voff<D>(vc, ld, wave, lane, valid);
      tile_dma<D>(qp, vc, ldsQ + slot * TL::BYTES, wave);
      tile_voff<D>(vc, ldo, wave, lane, valid);
      tile_dma<D>(op, vc, ldsO + slot * TL::BYTES, wave);
    }
    dma4_base(srow + (size_t)gi * T + ti * AB_KT, (uint32_t)(min(lane, valid - 1) * sizeof(float)), ldsS + slot * AB_KT * sizeof(float));
    if (++ti == nt) { ti = 0; gi++; }
  };
  if constexpr (D == 128) {
    // One wave has a SIMD to itself: beside its matrix instructions runs only what stands between them.  A 32x32x16 one keeps the matrix cores 32 cycles, a
    // tile's 64 of them 2048; a tile's other instructions (32 exponentials, 130 more of the vector ALU, 112 LDS reads, 9 transfers, 70 scalar ones) fill about
    // as many issue cycles and fit in their shadows if every slot gets its share.  Left to the compiler, half of dP's products ended up
    // behind all exponentials, and a tile took 4500 cycles.  So the matrix instructions are volatile, each is followed by its share, and all of it is pinned; fragments are
    // requested six products ahead (transposed ones eight); the next tile is published beside this one's dK products and its first fragments are read
    // there, so that no tile begins with a wait.  The same bits as in phases.  The whole backward pass (us, before and after): 32:8 heads x 4096 tokens 492 -> 465, 8:1 x
    // 8192 497 -> 473, 4:1 x 4096 queries over 12288 keys 330 -> 305, 2 x 2048 x 8 heads 81.4 -> 72.5, 4:1 x 4096 92 -> 88; sequences of one tile pay for the longer
    // start (four of 64 tokens 9.8 -> 10.3).  (Accumulators that start from the rows' delta save the 32 subtractions, 0.6 % of these, and
    // round at delta's scale on the way: a score gradient that cancels loses the small terms.)
    static_assert(AB_KT == 64 && AB_RING == 3, "slots below");
    constexpr int KS = D / 16, OFF1 = AB_RING * TL::BYTES;
    const lds_char* dir[KS];
    const lds_char* t0[D / 32];
    const lds_char* t1[D / 32];
    const lds_char* stp = sm + 2 * AB_RING * TL::BYTES + 4 * kg * sizeof(float);  // statistics of the lane's rows
#pragma unroll
    for (int ks = 0; ks < KS; ks++) dir[ks] = sm + fa.kdir[ks];
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) { t0[dt] = sm + fa.tr0[dt]; t1[dt] = sm + fa.tr1[dt]; }
    bf16x8 fr[4][2];         // score fragments of four k-steps
    bf16x8 tr[3][D / 32];    // transposed fragments of three groups of 16 rows: dO's groups are 0-3, Q's 4-7
    bf16x8 pf[2];            // packed P (groups 0-3), then dS (4-7)
    f32x4 lv[8], dl[8];      // log sums and delta of rows 32*mt + 8*q4 + 4*kg + e of the tile at [4*mt + q4]
    f32x16 st[2], dp[2];
    auto row_stat = [&](int ring, int x) { return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>(stp + ring + x * 32); };
    auto frag = [&](int step, int mt) {  // k-step `step` of the tile's S products, from KS on of its dP products
      fr[step & 3][mt] = lds_frag(dir[step & (KS - 1)], (step < KS ? 0 : OFF1) + mt * 32 * TL::LD * 2);
    };
    auto trfrag = [&](int group, int dt) { tr[group % 3][dt] = lds_frag_tr(t0[dt], t1[dt], (group < 4 ? OFF1 : 0) + (group & 3) * 16 * TL::LD * 2); };
    auto pack2 = [&](int group, int e) {  // elements 2e, 2e+1 of the group's fragment
      const f32x16& t = st[(group & 3) >> 1];
      pf[group & 1][2 * e] = (bf16_t)t[8 * (group & 1) + 2 * e];
      pf[group & 1][2 * e + 1] = (bf16_t)t[8 * (group & 1) + 2 * e + 1];
    };
    auto pack_share = [&](int group, int i) {  // beside the i-th product of the group before: none beside the last, a product later than the vector ALU writes
      if (i == 0) { pack2(group, 0); pack2(group, 1); }
      else if (i < 3) pack2(group, i + 1);
    };
    issue(0);
    if (f0 + 1 < f1) issue(1);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) asm volatile("" : "+a"(kf[ks]), "+a"(vf[ks]));
    const uint32_t ldsQw = ldsQ + wave * (TL::IPW * 1024), tile_bytes = TL::BYTES;
    const int ragged_ti = (seq - q0) % AB_KT != 0 ? nt - 1 : nt;  // the tile of each head that is not whole
    int slot = 0;
    const char *qp, *op, *sp;  // of the tile to transfer next
    auto sources = [&]() {
      qp = qbase + ti * qstride + gi * (D * sizeof(bf16_t));
      op = obase + ti * ostride + gi * (D * sizeof(bf16_t));
      sp = reinterpret_cast<const char*>(srow + (size_t)gi * T + ti * AB_KT);
    };
    sources();
    if (f0 + 1 < f1) dma_wait<2 * TL::IPW + 1>(); else dma_wait<0>();
    __syncthreads();
#pragma unroll
    for (int step = 0; step < 3; step++) { frag(step, 0); frag(step, 1); }
    for (int f = f0; f < f1; f++) {
      const int next = slot == AB_RING - 1 ? 0 : slot + 1, free_slot = slot == 0 ? AB_RING - 1 : slot - 1;
      const int step_tile = (next - slot) * TL::BYTES, step_stat = (next - slot) * AB_KT * (int)sizeof(float);
      asm volatile("s_barrier" ::: "memory");  // every wave is done with tile f-1: its slot is filled next
      const int qb = q0 + tc * AB_KT;
      if (++tc == nt) tc = 0;
      const bool more = f + 2 < f1, idle = qb + AB_KT - 1 < jw;  // idle: every query of the tile precedes every key of this wave
      const bool beside = more && !idle && ti != ragged_ti;
      if (more && !beside) { issue(free_slot); sources(); }
      auto publish = [&]() {  // tile f+1, whose transfers are followed by tile f+2's
        if (more) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * TL::IPW + 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
      };
      auto shift_dir = [&]() {
#pragma unroll
        for (int ks = 0; ks < KS; ks++) dir[ks] += step_tile;
      };
      auto shift_tr = [&]() {
#pragma unroll
        for (int dt = 0; dt < D / 32; dt++) { t0[dt] += step_tile; t1[dt] += step_tile; }
      };
      slot = next;
      if (idle) {
        publish();
        shift_dir();
        shift_tr();
        stp += step_stat;
#pragma unroll
        for (int step = 0; step < 3; step++) { frag(step, 0); frag(step, 1); }
        continue;
      }
      auto scores = [&](auto transfers) {
        constexpr bool TRANSFERS = decltype(transfers)::value;
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < 16; i++) {
          if (i < 2) mfma_first(st[i & 1], fr[(i >> 1) & 3][i & 1], kf[i >> 1]);
          else mfma_next(st[i & 1], fr[(i >> 1) & 3][i & 1], kf[i >> 1]);
          frag((i >> 1) + 3, i & 1);
          if (i < 8) dl[i] = row_stat(AB_RING * AB_KT * sizeof(float), i);
          else lv[i - 8] = row_stat(0, i - 8);
          if (TRANSFERS) {
            if (i == 2) m = dma_lds(ldsQw + free_slot * tile_bytes);
            if (i == 6) m = dma_lds(ldsQw + free_slot * tile_bytes + AB_RING * tile_bytes);
            if (i >= 2 && i < 6) dma16_at(m, qp, vq[i - 2], (i - 2) * 1024);
            if (i >= 6 && i < 10) dma16_at(m, op, vo[i - 6], (i - 6) * 1024);
            if (i == 10) dma4_base(sp, lane * sizeof(float), ldsS + free_slot * AB_KT * sizeof(float));
            if (i == 12) {
              qp += qstride;
              op += ostride;
              sp += AB_KT * sizeof(float);
            }
          }
          AB_PIN();
        }
      };
      if (beside) {
        scores(std::true_type{});
        if (++ti == nt) { ti = 0; gi++; sources(); }
      } else {
        scores(std::false_type{});
      }
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const int ks = i >> 1, mt = i & 1;
        if (ks == 0) mfma_first(dp[mt], fr[KS & 3][mt], vf[0]);
        else mfma_next(dp[mt], fr[(ks + KS) & 3][mt], vf[ks]);
        if (ks + 3 < KS) frag(ks + KS + 3, mt);
        if (i >= 8) trfrag((i - 8) >> 2, i & 3);
        if (i >= 2) {  // P from S, 32 values over 14 slots
#pragma unroll
          for (int x = (i - 2) * 32 / 14; x < (i - 1) * 32 / 14; x++) st[x >> 4][x & 15] = fast_exp2(fmaf(st[x >> 4][x & 15], scale_log2, -lv[x >> 2][x & 3]));
        }
        AB_PIN();
      }
      if (qb < jw + 32 || qb + AB_KT > seq) {  // diagonal tile, or rows past the end of the sequence
        const int first = qb + 4 * kg;
        const uint32_t rows = (uint32_t)max(seq - jk, 0);
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
          for (int r = 0; r < 16; r++) {
            st[mt][r] = (uint32_t)(first + mt * 32 + 8 * (r >> 2) + (r & 3) - jk) < rows ? st[mt][r] : 0.f;
            if ((r & 3) == 3) AB_PIN();
          }
      }
#pragma unroll
      for (int e = 0; e < 4; e++) pack2(0, e);
      frag_settle(pf[0]);
      // dV^T += dO^T P; a group of P, once packed, becomes dS = P (dP - delta) in place
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const int g = i >> 2, dt = i & 3;
        mfma_grad(dvt[dt], tr[g % 3][dt], pf[g & 1]);
        trfrag(g + 2, dt);
#pragma unroll
        for (int x = 8 * g + 2 * dt; x < 8 * g + 2 * dt + 2; x++) st[x >> 4][x & 15] *= dp[x >> 4][x & 15] - dl[x >> 2][x & 3];
        pack_share(g + 1, dt);
        if (i == 8) shift_dir();
        AB_PIN();
      }
      // dK^T += Q^T dS
#pragma unroll
      for (int i = 0; i < 16; i++) {
        const int g = 4 + (i >> 2), dt = i & 3;
        mfma_grad(dkt[dt], tr[g % 3][dt], pf[g & 1]);
        if (g < 6) trfrag(g + 2, dt);
        if (g < 7) pack_share(g + 1, dt);
        if (i == 8) publish();
        if (i == 9) shift_tr();
        if (i >= 10) frag((i - 10) >> 1, i & 1);
        AB_PIN();
      }
      stp += step_stat;
    }
  } else {
    issue(0);
    if (f0 + 1 < f1) issue(1);
    int slot = 0;
    for (int f = f0; f < f1; f++, slot = slot == AB_RING - 1 ? 0 : slot + 1) {
      if (f + 1 < f1) dma_wait<2 * TL::IPW + 1>(); else dma_wait<0>();
      __syncthreads();
      if (f + 2 < f1) issue(slot == 0 ? AB_RING - 1 : slot - 1);
      const int qb = q0 + tc * AB_KT;
      if (++tc == nt) tc = 0;
      if (qb + AB_KT - 1 < jw) continue;  // every query of the tile precedes every key of this wave
      TilePtrs<D> Qp, Op;
      Qp.set(sm + slot * TL::BYTES, fa);
      Op.set(sm + (AB_RING + slot) * TL::BYTES, fa);
      const float* ls = lse_s + slot * AB_KT;
      const float* ds = del_s + slot * AB_KT;
      f32x4 lv[8];  // rows 32*mt + 8*q4 + 4*kg + e of the tile at [4*mt + q4]
  #pragma unroll
      for (int x = 0; x < 8; x++) lv[x] = *reinterpret_cast<const f32x4*>(ls + 8 * x + 4 * kg);
      f32x16 st[2], dp[2];
      // P from S beside the dP products
      score_tiles2<D, AB_RING * TL::BYTES, 3>(st, Qp, kf, dp, vf, [&](int j) {
        constexpr int N = 8 / (D / 16);
  #pragma unroll
        for (int i = 0; i < N; i++) {
          const int x = j * N + i, mt = x >> 2, q4 = x & 3;
  #pragma unroll
          for (int e = 0; e < 4; e++) st[mt][4 * q4 + e] = fast_exp2(fmaf(st[mt][4 * q4 + e], scale_log2, -lv[x][e]));
        }
      });
      TrFrags<D> fr;
      tr_fetch<D>(fr, Op, 0);
  #pragma unroll
      for (int x = 0; x < 8; x++) lv[x] = *reinterpret_cast<const f32x4*>(ds + 8 * x + 4 * kg);
      if (qb < jw + 32 || qb + AB_KT > seq) {  // diagonal tile, or rows past the end of the sequence
        // One comparison a row, four rows at a time: two a row, all ahead of the selects, held 64 scalar registers at D = 64, and the
        // loop's own scalars (bases, strides, the head and tile to fetch next) were fetched from vector lanes in every tile (91 spilled: 32:4 heads x 1200
        // tokens, the whole backward pass, 65 us; now none, 56.  2 x 1000 69 -> 65, 8:1 x 4096 104 -> 97).
        const int first = qb + 4 * kg;
        const uint32_t rows = (uint32_t)max(seq - jk, 0);
  #pragma unroll
        for (int mt = 0; mt < 2; mt++)
  #pragma unroll
          for (int r = 0; r < 16; r++) {
            st[mt][r] = (uint32_t)(first + mt * 32 + 8 * (r >> 2) + (r & 3) - jk) < rows ? st[mt][r] : 0.f;
            if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);
          }
      }
      // dV^T += dO^T P; once a quarter of P (8 registers of a tile) is packed for its products, it is turned
      // into dS = P (dP - delta) in place while those products run; then dK^T += Q^T dS.
      acc_tile_tr<D, true, AGPR>(dvt, fr, Op, st, Qp, [&](int g) {
  #pragma unroll
        for (int r = 8 * (g & 1); r < 8 * (g & 1) + 8; r++) st[g >> 1][r] *= dp[g >> 1][r] - lv[4 * (g >> 1) + (r >> 2)][r & 3];
      });
      acc_tile_tr<D, false, AGPR>(dkt, fr, Qp, st, Qp, [](int) {});
    }
  }
  acc_settle<AGPR>(dkt);
  acc_settle<AGPR>(dvt);
  __syncthreads();  // every wave is done with the Q/dO rings: their LDS serves the output turn (dK, then dV)
  auto dk_quad = [&](int dt, int q4) {
    return f32x4{dkt[dt][4 * q4] * scale, dkt[dt][4 * q4 + 1] * scale, dkt[dt][4 * q4 + 2] * scale, dkt[dt][4 * q4 + 3] * scale};
  };
  auto dv_quad = [&](int dt, int q4) { return f32x4{dvt[dt][4 * q4], dvt[dt][4 * q4 + 1], dvt[dt][4 * q4 + 2], dvt[dt][4 * q4 + 3]}; };
  if (cm.chunks > 1) {
    float* rows = part + ((((size_t)b * nkv + hk) * pairs + cm.pair) * 128 + wave * 32) * (2 * D);
    float* reg = reinterpret_cast<float*>(smem) + wave * (32 * D);
    wave_rows_out_f32<D>(reg, lane, dk_quad, [&](int r) { return rows + (size_t)r * (2 * D); });
    __builtin_amdgcn_wave_barrier();
    wave_rows_out_f32<D>(reg, lane, dv_quad, [&](int r) { return rows + (size_t)r * (2 * D) + D; });
  } else {
    bf16_t* reg = reinterpret_cast<bf16_t*>(smem) + wave * (32 * D);
    wave_rows_out_bf16<D>(reg, lane, dk_quad,
                          [&](int r) { return jw + r < seq ? g.dkv + (ktok0 + jw + r) * g.lddkv + (size_t)hk * D : nullptr; });
    __builtin_amdgcn_wave_barrier();
    wave_rows_out_bf16<D>(reg, lane, dv_quad,
                          [&](int r) { return jw + r < seq ? g.dkv + (ktok0 + jw + r) * g.lddkv + (size_t)(nkv + hk) * D : nullptr; });
  }
}

// One launch for both halves of the backward pass, used when every query head has a key/value head of its own.  Alone,
// each half leaves compute units idle while its longest blocks finish; in one grid the dQ units fill the gaps of the
// dK/dV units and the other way round (measured on MI355X at 2 x 2048 tokens, 8 heads: 122 -> 94 us).  With grouped
// heads the same merge measured slower than two launches (4096 tokens, 4:1 heads: 128 -> 145 us; 8192 tokens, 8:1:
// 594 -> 652 us), so those shapes keep two launches.  Launch index -> (head, unit): units of the two kinds alternate, each kind
// heaviest first, the dK/dV unit (the dearer one) leading; once the shorter list is used up the rest of the longer
// follows.  grid ((pairs_q + pairs_k) * nq * batch).
template <int D>
__global__ __launch_bounds__(AB_THREADS) void attn_bwd_bf16_kernel(const AttnGeom gq, const AttnGeom gk, const bf16_t* __restrict__ qkv,
                                                                   const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                                                                   const float* __restrict__ lse, const float* __restrict__ lse2,
                                                                   const float* __restrict__ delta, bf16_t* __restrict__ dqkv,
                                                                   float* __restrict__ part_q, float* __restrict__ part_kv, int pairs_q,
                                                                   int pairs_k, int T, float scale, float scale_log2) {
  const int hb = blockIdx.x % gq.nq_all, u = blockIdx.x / gq.nq_all, both = 2 * min(pairs_q, pairs_k);
  int idx;
  bool dkv;
  if (u < both) { dkv = (u & 1) == 0; idx = u >> 1; }
  else { dkv = pairs_k > pairs_q; idx = u - both / 2; }
  if (dkv) attn_bwd_dkv_block<D>(idx * gk.nq_all + hb, gk, qkv, dout, lse2, delta, part_kv, pairs_k, T, scale, scale_log2);
  else attn_bwd_dq_block<D, AB_RING>(idx * gq.nq_all + hb, gq, qkv, o, dout, lse, nullptr, nullptr, dqkv, part_q, pairs_q, T, scale, scale_log2);
}
// The two halves as launches of their own (dQ first: it stores the row statistics the dK/dV blocks read).
template <int D>
__global__ __launch_bounds__(AB_THREADS, 2) void attn_bwd_dq_bf16_kernel(const AttnGeom g, const bf16_t* __restrict__ qkv,
                                                                      const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                                                                      const float* __restrict__ lse, float* __restrict__ lse2,
                                                                      float* __restrict__ delta, bf16_t* __restrict__ dqkv,
                                                                      float* __restrict__ part, int pairs, int T, float scale, float scale_log2) {
  attn_bwd_dq_block<D, dq_ring(D)>((int)blockIdx.x, g, qkv, o, dout, lse, lse2, delta, dqkv, part, pairs, T, scale, scale_log2);
}
template <int D>
__global__ __launch_bounds__(AB_THREADS) void attn_bwd_dkv_bf16_kernel(const AttnGeom g, const bf16_t* __restrict__ qkv,
                                                                       const bf16_t* __restrict__ dout, const float* __restrict__ lse2,
                                                                       const float* __restrict__ delta, float* __restrict__ part,
                                                                       int pairs, int T, float scale, float scale_log2) {
  attn_bwd_dkv_block<D>((int)blockIdx.x, g, qkv, dout, lse2, delta, part, pairs, T, scale, scale_log2);
}

// Per-row statistics of the backward pass for the dK/dV blocks: delta[h,t] = sum_c dO[t,h,c] O[t,h,c] and
// lse2[h,t] = lse[h,t] log2(e).  The sum runs in the order the dQ blocks use for their own copy (two halves of the row,
// each 8 elements out of every 16, one fused multiply-add per element, halves added last), so both kernels work with
// the same numbers.  Two neighbouring lanes per (token, head), one for each half, in blocks of one wave: bound by one round of loads.  (A thread
// per row in blocks of 256: 528 tokens, 4 heads 6.6 us, now 2.8.)
template <int D>
__global__ __launch_bounds__(64) void attn_bwd_prep_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ dout,
                                                           const float* __restrict__ lse, float* __restrict__ lse2,
                                                           float* __restrict__ delta, int T, int nq) {
  const size_t i = (size_t)blockIdx.x * 32 + (threadIdx.x >> 1);
  if (i >= (size_t)T * nq) return;
  const int kg = threadIdx.x & 1, h = (int)(i % nq);
  const size_t t = i / nq, at = (size_t)h * T + t;
  const bf16_t* orow = o + (t * nq + h) * D + kg * 8;
  const bf16_t* drow = dout + (t * nq + h) * D + kg * 8;
  const float l = lse[at];
  bf16x8 a[D / 16], b[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    a[ks] = *reinterpret_cast<const bf16x8*>(drow + ks * 16);
    b[ks] = *reinterpret_cast<const bf16x8*>(orow + ks * 16);
  }
  float half = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++)
#pragma unroll
    for (int e = 0; e < 8; e++) half = fmaf((float)a[ks][e], (float)b[ks][e], half);
  const float other = __shfl_xor(half, 1, 64);
  if (kg == 0) {
    delta[at] = half + other;
    lse2[at] = l * LOG2E;
  }
}

// dk,dv[token][kv head] = sum over the chunks of the token's key block (ascending) of the float32 partials, where it has several.
// grid (32*ceil(seq/128), nkv, batch), 256 threads: a block owns 4 rows of a key block, thread = (key row, 4
// columns of [dK | dV]).
template <int D>
__device__ __forceinline__ void attn_bwd_group_reduce_block(int bx, int by, int bz, const float* __restrict__ part, const AttnGeom& g,
                                                            int pairs) {
  const int seq = g.seq, nkv = g.nkv;
  const int i = bx >> 5, r0 = (bx & 31) * 4, hk = by, b = bz;
  const int ch = chunks_of(g.grp * dkv_tiles(i, seq, g.q_off), g.ch);
  if (ch == 1) return;  // written by its only chunk
  const int base = wave_sum(0, i, [&](int k) { return chunks_of(g.grp * dkv_tiles(k, seq, g.q_off), g.ch); });
  const float* p0 = part + (((size_t)b * nkv + hk) * pairs + base) * 128 * (2 * D);
  for (int e = threadIdx.x; e < 4 * 2 * D / 4; e += 256) {
    const int row = r0 + e / (2 * D / 4), c4 = (e % (2 * D / 4)) * 4;
    if (i * 128 + row >= seq) continue;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < ch; c++) s += __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p0 + ((size_t)c * 128 + row) * (2 * D) + c4));
    bf16x4 o = {(bf16_t)s[0], (bf16_t)s[1], (bf16_t)s[2], (bf16_t)s[3]};
    bf16_t* dst = g.dkv + ((size_t)b * seq + i * 128 + row) * g.lddkv + (c4 < D ? (size_t)hk * D + c4 : (size_t)(nkv + hk) * D + (c4 - D));
    *reinterpret_cast<bf16x4*>(dst) = o;
  }
}

// Both merges in one launch (they are independent, short and bandwidth-bound): the first nb_q blocks are the
// (x, y, z) = (16 * query blocks, nq, batch) grid of the dQ merge, the rest the (32 * key blocks, nkv, batch) grid of
// the dK/dV merge; either part may be empty.
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_reduce_kernel(const float* __restrict__ part_q, bf16_t* __restrict__ dqkv, int pairs_q,
                                                              int ch_q, float scale, unsigned nb_q, unsigned gqx, unsigned gqy,
                                                              const float* __restrict__ part_kv, const AttnGeom g, int pairs_k,
                                                              unsigned gkx, unsigned gky) {
  unsigned id = blockIdx.x;
  if (id < nb_q) {
    attn_bwd_dq_reduce_block<D>((int)(id % gqx), (int)(id / gqx % gqy), (int)(id / (gqx * gqy)), part_q, dqkv, g.seq, g.q_off, g.nq,
                                g.nkv, pairs_q, ch_q, scale);
  } else {
    id -= nb_q;
    attn_bwd_group_reduce_block<D>((int)(id % gkx), (int)(id / gkx % gky), (int)(id / (gkx * gky)), part_kv, g, pairs_k);
  }
}

// ------------------------------------------------------------------------------------ host side
template <typename K>
static int set_lds(K kernel, size_t bytes) {
  DH_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
  return DH_OK;
}

static int attn_num_cus() {  // of the current device
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

// Chunk length of a backward launch.  The blocks of a launch are (block of 128 positions, chunk) units times heads * batch, launched heaviest
// first; what a chunk length takes is simulated and the best one taken.  The hardware hands blocks to the 8 dies in turn and, on a die, to its 4
// shader engines in turn, none before the one ahead of it: a block waits for a unit of its engine though others are
// free.  (That order fits what chunk lengths measure: dK/dV of 8 heads x 8192 tokens on one key/value head, 136 / 140 / 144 tiles a chunk
// 535 / 504 / 509 us for the whole backward pass, where the first free unit would make 136 the best.)  The constants are measured on MI355X
// (microseconds at D = 128; D = 64 below): a block's tile with two blocks on its unit 2.2 for dQ (0.55 of that with one), dK/dV, alone on its
// unit, 2.0; a block beyond its tiles 3 (dQ), 7 (dK/dV; 9 where they share a launch), with a partial dK/dV result 2 more; partial results are written and
// read back at 2-5 MB per microsecond, by a launch of its own that takes 4-12 and that dK/dV's share with dQ's.
// Where every query head has a key/value head of its own, dQ and dK/dV units fill one launch, alternating, and are cut alike, up to the
// longest of either kind: behind a key buffer the query blocks' rows are far longer than the key blocks' columns (4 heads x 189 queries over 7997 keys: 125
// and 3 tiles), and lengths up to the columns' alone left them whole (176 us, cut into 14 tiles 36).
enum { PICK_FWD, PICK_DQ, PICK_DKV, PICK_BOTH };
struct PickKey {
  int kind, seq, q_off, nq_all, d, grp, merged, cus;
  bool operator<(const PickKey& o) const {
    return std::tie(kind, seq, q_off, nq_all, d, grp, merged, cus) < std::tie(o.kind, o.seq, o.q_off, o.nq_all, o.d, o.grp, o.merged, o.cus);
  }
};
struct LaunchUnit { int tiles; bool part; };  // part: it stores a partial result
// Tiles of the units of a dK/dV launch, in launch order (see map_dkv).
static std::vector<LaunchUnit> dkv_units(int seq, int q_off, int grp, int ch) {
  std::vector<LaunchUnit> units, rest;
  for (int i = 0; i < (seq + 127) / 128; i++) {
    const int t = grp * dkv_tiles(i, seq, q_off);
    units.insert(units.end(), t / ch, {ch, t > ch});
    if (t % ch) rest.push_back({t % ch, t > ch});
  }
  std::stable_sort(rest.begin(), rest.end(), [](const LaunchUnit& a, const LaunchUnit& b) { return a.tiles > b.tiles; });
  units.insert(units.end(), rest.begin(), rest.end());
  return units;
}
struct LaunchModel {
  int resident;       // blocks a unit holds
  double tile, alone, ovh, part, us_per_byte, merge;  // part: what a partial result adds to a block
  bool tail;          // a block whose neighbour on the unit is through goes on faster
};
static LaunchModel launch_model(int kind, int d) {
  // D = 64: fitted with the tail to ten shapes, 600 to 7000 tokens on 8 to 32 heads; the length taken is 0.3 % behind the best one on average.  Without it (and
  // with the constants of D = 128) whole rows, whose longest blocks end by themselves, looked longer than they are: 16:2 heads x 5000 tokens
  // dQ in chunks of 68 tiles 120 us, whole 102.
  if (kind == PICK_DQ && d == 64) return {2, 1.1, 0.65, 3.0, 0.0, 1 / 3.0e6, 4.0, true};
  if (kind == PICK_DQ) return {2, 2.2, 0.55, 3.0, 0.0, 1 / 5.0e6, 4.0, false};
  // dK/dV of grouped heads: fitted to 60 shapes, 100 to 7000 queries of up to 64 heads, keys before them or not: the length taken is 0.9 % behind the best one on
  // average, 3.7 with one set of constants for this and the shared launch.  Those priced a cut so high that the few blocks of short sequences walked their
  // whole head group one tile after the other (whole pass, 4:2 heads x 224 tokens 32.6 us, in chunks of two tiles 26; D = 64, 32:8 x 145 27 and 20; a block
  // per query head 29 and 22).
  if (kind == PICK_DKV && d == 64) return {2, 1.6, 0.92, 2.2, 1.0, 1 / 1.5e6, 5.0, false};
  if (kind == PICK_DKV) return {1, 2.0, 1.0, 7.0, 2.0, 1 / 2.0e6, 4.0, false};
  // The shared launch at D = 64: fitted to 48 shapes, 0.9 % behind the best length on average (2.9 with overheads scaled from D = 128, which cut
  // rows that are faster whole: 8 heads x 2 x 1660 tokens 50 us, whole 45).
  if (d == 64) return {2, 1.73, 0.76, 8.0, 0.25, 1 / 1.1e6, 5.6, false};
  return {1, 2.0, 1.0, 9.0, 0.0, 1 / 4.0e6, 12.0, false};
}
// simulate_launch for blocks that share a unit two by two, each as fast as the unit's other block lets it be.
static double simulate_tail(const LaunchModel& m, const std::vector<LaunchUnit>& units, int heads) {
  struct Unit { double at, left[2]; int n, version; };  // work left of its n blocks at time `at`, in us of a block alone
  struct Event {
    double end;
    int engine, unit, version;
    bool operator<(const Event& o) const { return end > o.end; }
  };
  const int per = std::max(1, attn_num_cus() / 32);
  std::vector<Unit> unit(32 * per, Unit{0.0, {0.0, 0.0}, 0, 0});
  std::priority_queue<Event> ends;
  const long long all = (long long)units.size() * heads;
  long long next[8];  // of the blocks of a die
  for (int die = 0; die < 8; die++) next[die] = die;
  auto rate = [&](const Unit& u) { return u.n > 1 ? m.alone : 1.0; };
  auto advance = [&](Unit& u, double now) {
    for (int i = 0; i < u.n; i++) u.left[i] -= rate(u) * (now - u.at);
    u.at = now;
  };
  auto expect = [&](int engine, int c) {
    Unit& u = unit[engine * per + c];
    u.version++;
    if (u.n > 0) ends.push({u.at + (u.n > 1 ? std::min(u.left[0], u.left[1]) : u.left[0]) / rate(u), engine, c, u.version});
  };
  auto place = [&](int die, double now) {  // the die's next blocks, in order, until one finds its engine full
    for (; next[die] < all; next[die] += 8) {
      const int engine = die * 4 + (int)((next[die] >> 3) & 3);
      int c = 0;
      for (int i = 1; i < per; i++) if (unit[engine * per + i].n < unit[engine * per + c].n) c = i;
      Unit& u = unit[engine * per + c];
      if (u.n >= 2) return;
      advance(u, now);
      u.left[u.n++] = units[next[die] / heads].tiles * m.tile * m.alone + m.ovh;
      expect(engine, c);
    }
  };
  for (int die = 0; die < 8; die++) place(die, 0.0);
  double now = 0.0;
  while (!ends.empty()) {
    const Event e = ends.top();
    ends.pop();
    Unit& u = unit[e.engine * per + e.unit];
    if (e.version != u.version) continue;
    now = e.end;
    advance(u, now);
    int n = 0;
    for (int i = 0; i < u.n; i++) if (u.left[i] > 1e-6) u.left[n++] = u.left[i];
    u.n = n;
    expect(e.engine, e.unit);
    place(e.engine / 4, now);
  }
  return now;
}
// units: those of one head, in launch order.
static double simulate_launch(const LaunchModel& m, const std::vector<LaunchUnit>& units, int heads) {
  typedef std::priority_queue<double, std::vector<double>, std::greater<double>> Queue;
  const int cus = attn_num_cus();
  Queue unit[8][4];
  double ahead[8] = {};
  for (auto& die : unit) for (Queue& q : die) for (int i = 0; i < std::max(1, cus * m.resident / 32); i++) q.push(0.0);
  const long long all = (long long)units.size() * heads;
  const double tile = m.tile * (all <= cus ? m.alone : 1.0);
  double makespan = 0.0;
  long long k = 0;
  for (const LaunchUnit& u : units)
    for (int h = 0; h < heads; h++, k++) {
      Queue& q = unit[k & 7][(k >> 3) & 3];
      double& start = ahead[k & 7];
      start = std::max(start, q.top());
      q.pop();
      const double end = start + u.tiles * tile + m.ovh + (u.part ? m.part : 0.0);
      q.push(end);
      makespan = std::max(makespan, end);
    }
  return makespan;
}
// heads: heads * batch of the launch (query heads; key/value heads for dK/dV); grp: query heads of a key/value head; merged: partial results are
// added by a launch that is there anyway.
static int pick_bwd_chunk(int kind, int seq, int q_off, int heads, int d, int grp, bool merged) {
  LaunchModel m = launch_model(kind, d);
  if (merged) m.merge = 0.0;
  const int nblk = (seq + 127) / 128, qb0 = q_off / 128, most_q = dq_tiles(nblk - 1, seq), most_k = grp * dkv_tiles(0, seq, q_off);
  const int max_tiles = kind == PICK_DQ ? most_q : kind == PICK_DKV ? most_k : std::max(most_q, most_k);
  const long long slots = (long long)attn_num_cus() * m.resident;
  const long long all_blocks = (long long)nblk * heads, before_q = (long long)qb0 * heads;  // before_q: short key blocks ahead of the queries
  int best = AB_WHOLE;
  double best_t = 1e300;
  auto consider = [&](int ch) {
    const long long count = (kind >= PICK_DKV ? total_pairs_dkv(seq, q_off, ch, grp) : 0) + (kind != PICK_DKV ? total_pairs_dq(seq, q_off, ch) : 0);
    if (count * heads > 16 * slots + (kind == PICK_BOTH ? before_q : 0) && ch < AB_WHOLE) return;  // so many rounds need no chunks as short
    std::vector<LaunchUnit> units, q_units;
    double bytes = 0;  // of partial results, per head
    if (kind >= PICK_DKV) {
      units = dkv_units(seq, q_off, grp, ch);
      for (int i = 0; i < nblk; i++) { const int n = chunks_of(grp * dkv_tiles(i, seq, q_off), ch); bytes += n > 1 ? n * 2.0 * d : 0; }
    }
    if (kind != PICK_DKV)
      for (int i = nblk - 1; i >= qb0; i--) {
        const int tiles = dq_tiles(i, seq), n = chunks_of(tiles, ch);
        for (int c = 0; c < n; c++) q_units.push_back({std::min(ch, tiles - c * ch), n > 1});
        bytes += n > 1 ? n * (double)d : 0;
      }
    if (kind == PICK_BOTH) {  // as attn_bwd_bf16_kernel takes them
      std::vector<LaunchUnit> all;
      for (size_t k = 0; k < std::max(units.size(), q_units.size()); k++) {
        if (k < units.size()) all.push_back(units[k]);
        if (k < q_units.size()) all.push_back(q_units[k]);
      }
      units = all;
    } else if (kind != PICK_DKV) {
      units = q_units;
    }
    const double t = (m.tail ? simulate_tail(m, units, heads) : simulate_launch(m, units, heads)) + (bytes > 0 ? bytes * heads * 128 * sizeof(float) * m.us_per_byte + m.merge : 0.0);
    if (t < best_t) { best_t = t; best = ch; }
  };
  if (all_blocks - (kind == PICK_BOTH ? before_q : 0) < 8 * slots && all_blocks < 32 * slots && nblk <= 1024) {
    consider(AB_WHOLE);
    const int least = kind == PICK_DKV ? 1 : 2;  // dQ: even, so that every wave sees a chunk's first tile
    for (int c = 2 * least; c < max_tiles; c += std::max(least, c / 32 * least)) consider(c);
  }
  return best;
}

// Chunk length of a forward launch: a few lengths and a plain list schedule (1.45 us a tile at D = 128, the loop in phases, 3 a block, partial results there
// and back at 2 MB per microsecond and 12 for their launch); where splitting pays, then the shortest length whose blocks are all resident
// at once, two a unit (4 heads x 4096 tokens, 16 -> 10 tiles 48 -> 42 us; one block more than fits costs a second round).
// The model above finds shorter launches (3 x 1365 tokens, 4 heads, 29 -> 24 us; 4 heads x 8192 at D = 64 89 -> 61 us), but other lengths
// add a row's partial results over other ranges of keys, and then gradients that are all rounding come out as other noise (the router's,
// exactly zero where a token's two experts hold the same weights): the lengths stay, also where they are the 8 tiles that the loop in phases takes
// (fwd_pinned).
static int pick_fwd_chunk(int seq, int q_off, int heads, int d) {
  const int nblk = (seq + 127) / 128, qb0 = q_off / 128, slots = attn_num_cus();
  auto units_of = [&](int ch) { return (long long)total_pairs_dq(seq, q_off, ch); };  // the tiles dQ walks
  int best = AB_WHOLE;
  double best_t = 1e300;
  for (int ch : {4, 8, 16, 32, 64, AB_WHOLE}) {
    if (ch < AB_WHOLE && ch >= dq_tiles(nblk - 1, seq)) continue;
    std::priority_queue<double, std::vector<double>, std::greater<double>> free_at;
    for (int i = 0; i < slots; i++) free_at.push(0.0);
    double t = 0.0;
    for (int i = nblk - 1; i >= qb0; i--)
      for (int t0 = 0, tiles = dq_tiles(i, seq); t0 < tiles; t0 += ch)
        for (int h = 0; h < heads; h++) {
          const double end = free_at.top() + std::min(ch, tiles - t0) * (1.45 * d / 128.0) + 3.0;
          free_at.pop();
          free_at.push(end);
          t = std::max(t, end);
        }
    if (units_of(ch) > nblk - qb0) t += (double)units_of(ch) * (d + 2) * heads * 128 * sizeof(float) * (2.0 / 4.0e6) + 12.0;
    if (t < best_t) { best_t = t; best = ch; }
  }
  for (int ch = 8; ch < best && best < AB_WHOLE; ch += 2)
    if (units_of(ch) * heads <= 2 * slots) return ch;
  return best;
}

static int pick_chunk(int kind, int seq, int q_off, int heads, int d, int grp, bool merged = false) {
  static std::mutex mu;
  static std::map<PickKey, int> cache;
  const PickKey key{kind, seq, q_off, heads, d, grp, merged ? 1 : 0, attn_num_cus()};
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(key);
  if (it == cache.end())
    it = cache.emplace(key, kind == PICK_FWD ? pick_fwd_chunk(seq, q_off, heads, d) : pick_bwd_chunk(kind, seq, q_off, heads, d, grp, merged)).first;
  return it->second;
}

// Tiles per chunk of the forward kernel; 0 = blocks are not split.
static int fwd_chunk_tiles(int batch, int seq, int q_off, int nq, int d) {
  const int ch = pick_chunk(PICK_FWD, seq, q_off, nq * batch, d, 1);
  return ch >= AB_WHOLE ? 0 : ch;
}
// Tiles per chunk of the dQ and of the dK/dV kernel.
static void bwd_chunk_tiles(int batch, int seq, int q_off, int nq, int nkv, int d, int& ch_q, int& ch_k) {
  if (nq == nkv) {
    ch_q = ch_k = pick_chunk(PICK_BOTH, seq, q_off, nq * batch, d, 1);
    if (ch_k >= dkv_tiles(0, seq, q_off)) ch_k = AB_WHOLE;  // no key block is cut: none need look for its chunk (4 heads x 189 over 7997 keys 40 -> 36 us)
  } else {
    ch_q = pick_chunk(PICK_DQ, seq, q_off, nq * batch, d, 1);
    ch_k = pick_chunk(PICK_DKV, seq, q_off, nkv * batch, d, nq / nkv, total_pairs_dq(seq, q_off, ch_q) > (seq + 127) / 128 - q_off / 128);
  }
}

// The launchers take the queries' sequence length seq_q and q_off; kv == nullptr selects plain attention (keys and
// values in the packed qkv rows, gradients into the packed dqkv rows).
static int check_geom(int d, int q_off, const void* kv, int ldkv, int nkv) {
  if (d != 64 && d != 128) DH_FAIL(DH_ERR_SHAPE, "attention (bf16): head_dim %d must be 64 or 128", d);
  if (q_off < 0 || q_off % 128) DH_FAIL(DH_ERR_SHAPE, "attention (bf16): the query offset %d must be a non-negative multiple of 128", q_off);
  if (!kv && q_off) DH_FAIL(DH_ERR_INVALID_ARG, "attention (bf16): a query offset needs a key/value buffer");
  if (kv && (ldkv < 2 * nkv * d || ldkv % 8 || ((uintptr_t)kv & 15)))
    DH_FAIL(DH_ERR_SHAPE, "attention (bf16): key/value rows must hold 2*nkv*d elements, be a multiple of 8 long and 16-byte aligned");
  return DH_OK;
}

size_t dh_attn_fwd_bf16_ws_bytes(int batch, int seq_q, int q_off, int nq, int nkv, int d) {
  (void)nkv;
  if (batch * seq_q == 0) return 0;
  const int seq = q_off + seq_q, ch = fwd_chunk_tiles(batch, seq, q_off, nq, d);
  if (ch == 0) return 0;
  return (size_t)batch * nq * fwd_units(seq, q_off, ch) * 128 * ((size_t)d + 2) * sizeof(float);
}

// Whether the pipelined kernel takes a launch: units of few tiles spend longer in its start (the first tile's scores stand alone, twice the code is
// fetched) than its loop gains.  us, in phases and pipelined: 4:1 heads x 300 tokens (5 tiles) 9.3 and 9.7, 32:8 x 343 (6) 11.8 and 11.9,
// 8:2 x 1280 (chunks of 8) 23.1 and 23.6, 3 x 488 on 4:2 (8) 13.8 and 13.4, 4:1 x 4096 (chunks of 10) 36.6 and 35.6, 3968 35.3 and 34.4, 3 x 683 (11) 16.5 and 15.2.
static bool fwd_pinned(int d, int seq, int ch) { return d == 128 && (ch > 0 ? ch : fwd_tiles((seq + 127) / 128 - 1, seq)) >= 10; }
int dh_launch_attn_fwd_bf16(int batch, int seq_q, int nq, int nkv, int d, const bf16_t* qkv, const bf16_t* kv, int ldkv, int q_off,
                            bf16_t* o, float* lse, void* ws, size_t ws_bytes, hipStream_t stream) {
  int rc;
  if ((rc = check_geom(d, q_off, kv, ldkv, nkv))) return rc;
  if (batch * seq_q == 0) return DH_OK;
  const int seq = q_off + seq_q, T = batch * seq_q;
  AttnGeom g;
  g.seq = seq; g.q_off = q_off; g.nq = nq; g.nkv = nkv; g.dkv = nullptr; g.lddkv = 0; g.ch = 0; g.nq_all = nq * batch; g.grp = nq / nkv;
  if (kv) { g.kv = kv; g.ldkv = ldkv; } else { g.kv = qkv + (size_t)nq * d; g.ldkv = (nq + 2 * nkv) * d; }
  const int nblk = (seq + 127) / 128 - q_off / 128;  // blocks that hold queries
  int ch = fwd_chunk_tiles(batch, seq, q_off, nq, d);
  if (ch > 0 && (!ws || ws_bytes < dh_attn_fwd_bf16_ws_bytes(batch, seq_q, q_off, nq, nkv, d))) ch = 0;  // no room for partial results
  const int units = ch > 0 ? fwd_units(seq, q_off, ch) : nblk;
  float* part_o = (float*)ws;
  float* part_ml = ch > 0 ? part_o + (size_t)batch * nq * units * 128 * d : nullptr;
  dim3 cgrid(nblk * 8, nq, batch);
  const float sl2 = (float)(1.4426950408889634 / sqrt((double)d));
  static bool ready_dev[DH_MAX_DEVICES][3] = {};
  bool* ready = ready_dev[dh_device_index()];
  auto launch = [&](auto kernel, bool& set, int slots) -> int {
    const size_t lds = (size_t)slots * AB_KT * d * sizeof(bf16_t);
    if (!set) {
      if (int e = set_lds(kernel, lds)) return e;
      set = true;
    }
    kernel<<<(unsigned)units * nq * batch, AB_THREADS, lds, stream>>>(g, qkv, o, lse, T, sl2, ch, units, part_o, part_ml);
    DH_LAUNCH_CHECK();
    return DH_OK;
  };
  if (fwd_pinned(d, seq, ch)) rc = launch(attn_fwd_pinned_bf16_kernel, ready[0], AF_K_RING + AF_V_RING);
  else if (d == 128) rc = launch(attn_fwd_bf16_kernel<128>, ready[1], 2 * AF_RING);
  else rc = launch(attn_fwd_bf16_kernel<64>, ready[2], 2 * AF_RING);
  if (rc || ch == 0) return rc;
  if (d == 128) attn_fwd_combine_kernel<128><<<cgrid, 256, 0, stream>>>(seq, q_off, nq, ch, units, part_o, part_ml, o, lse, T);
  else attn_fwd_combine_kernel<64><<<cgrid, 256, 0, stream>>>(seq, q_off, nq, ch, units, part_o, part_ml, o, lse, T);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

// workspace: lse2[nq*T] floats; dK/dV partials [batch][nkv][pairs][128][2d] floats when some key block has more than one
// chunk; dQ partials [batch][nq][pairs][128][d] floats when some query block has
struct BwdLayout {
  size_t o_lse2, o_dkv, o_dq, total;
  int ch_q, ch_k, pq, pk;   // chunk lengths and (block, chunk) pair counts of the dQ and the dK/dV launch
  bool part_q, part_kv;     // whether the launch writes float32 partial results
};
static BwdLayout bwd_ws_layout(int batch, int seq_q, int q_off, int nq, int nkv, int d) {
  BwdLayout L;
  const size_t T = (size_t)batch * seq_q;
  const int seq = q_off + seq_q, nblk = (seq + 127) / 128;
  bwd_chunk_tiles(batch, seq, q_off, nq, nkv, d, L.ch_q, L.ch_k);
  L.pq = total_pairs_dq(seq, q_off, L.ch_q);
  L.pk = total_pairs_dkv(seq, q_off, L.ch_k, nq / nkv);
  L.part_q = L.pq > nblk - q_off / 128;
  L.part_kv = L.pk > nblk;
  size_t cur = 0;
  L.o_lse2 = cur; cur += dh_align_up(nq * T * sizeof(float), 256);
  L.o_dkv = cur; if (L.part_kv) cur += dh_align_up((size_t)batch * nkv * L.pk * 128 * 2 * d * sizeof(float), 256);
  L.o_dq = cur; if (L.part_q) cur += dh_align_up((size_t)batch * nq * L.pq * 128 * d * sizeof(float), 256);
  L.total = cur;
  return L;
}

size_t dh_attn_bwd_bf16_ws_bytes(int batch, int seq_q, int q_off, int nq, int nkv, int d) {
  return bwd_ws_layout(batch, seq_q, q_off, nq, nkv, d).total;
}

int dh_launch_attn_bwd_bf16(int batch, int seq_q, int nq, int nkv, int d, const bf16_t* qkv, const bf16_t* kv, int ldkv, int q_off,
                            const bf16_t* o, const bf16_t* dout, const float* lse, bf16_t* dqkv, bf16_t* dkv, int lddkv,
                            float* delta, void* ws, size_t ws_bytes, hipStream_t stream) {
  int rc;
  if ((rc = check_geom(d, q_off, kv, ldkv, nkv))) return rc;
  if (kv && (!dkv || lddkv < 2 * nkv * d || lddkv % 8 || ((uintptr_t)dkv & 15)))
    DH_FAIL(DH_ERR_SHAPE, "attention (bf16): the key/value gradient buffer must match the key/value buffer's layout rules");
  const int T = batch * seq_q, seq = q_off + seq_q;
  if (T == 0) return DH_OK;
  AttnGeom g;
  g.seq = seq; g.q_off = q_off; g.nq = nq; g.nkv = nkv;
  if (kv) { g.kv = kv; g.ldkv = ldkv; g.dkv = dkv; g.lddkv = lddkv; }
  else { g.kv = qkv + (size_t)nq * d; g.dkv = dqkv + (size_t)nq * d; g.ldkv = g.lddkv = (nq + 2 * nkv) * d; }
  const BwdLayout lay = bwd_ws_layout(batch, seq_q, q_off, nq, nkv, d);
  g.nq_all = nq * batch;
  g.grp = nq / nkv;
  AttnGeom gq_geom = g, gk_geom = g;
  gk_geom.nq_all = nkv * batch;
  gq_geom.ch = lay.ch_q;
  gk_geom.ch = lay.ch_k;
  if (!ws || ws_bytes < lay.total) DH_FAIL(DH_ERR_WORKSPACE_TOO_SMALL, "attn_bwd: workspace %zu < %zu bytes", ws_bytes, lay.total);
  float* lse2 = (float*)((char*)ws + lay.o_lse2);
  float* part_kv = lay.part_kv ? (float*)((char*)ws + lay.o_dkv) : nullptr;
  float* part_q = lay.part_q ? (float*)((char*)ws + lay.o_dq) : nullptr;
  const float sc = (float)(1.0 / sqrt((double)d)), sl2 = (float)(1.4426950408889634 / sqrt((double)d));
  const int nblk = (seq + 127) / 128, nblk_q = nblk - q_off / 128, pq = lay.pq, pk = lay.pk;
  dim3 gw((unsigned)(pq + pk) * nq * batch), gwq((unsigned)pq * nq * batch), gwk((unsigned)pk * nkv * batch), gq(nblk_q * 16, nq, batch),
      gk(nblk * 32, nkv, batch);
  const unsigned nb_q = part_q ? gq.x * gq.y * gq.z : 0, nb_k = part_kv ? gk.x * gk.y * gk.z : 0;
  const size_t lds_dq = 2 * dq_ring(d) * (size_t)AB_KT * d * 2, lds_dkv = 2 * AB_RING * ((size_t)AB_KT * d * 2 + AB_KT * sizeof(float));
  static bool ready_dev[DH_MAX_DEVICES][2] = {};
  bool* ready = ready_dev[dh_device_index()];
#define DH_ATTN_BWD(DD, IDX)                                                                                                   \
  do {                                                                                                                         \
    if (!ready[IDX]) {                                                                                                         \
      if ((rc = set_lds(attn_bwd_bf16_kernel<DD>, lds_dkv)) || (rc = set_lds(attn_bwd_dq_bf16_kernel<DD>, lds_dq)) ||          \
          (rc = set_lds(attn_bwd_dkv_bf16_kernel<DD>, lds_dkv))) return rc;                                                    \
      ready[IDX] = true;                                                                                                       \
    }                                                                                                                          \
    if (nq == nkv) {                                                                                                           \
      attn_bwd_prep_kernel<DD><<<(unsigned)(((size_t)T * nq + 31) / 32), 64, 0, stream>>>(o, dout, lse, lse2, delta, T, nq); \
      DH_LAUNCH_CHECK();                                                                                                       \
      attn_bwd_bf16_kernel<DD><<<gw, AB_THREADS, lds_dkv, stream>>>(gq_geom, gk_geom, qkv, o, dout, lse, lse2, delta, dqkv, part_q, \
                                                                   part_kv, pq, pk, T, sc, sl2);                               \
    } else {                                                                                                                   \
      attn_bwd_dq_bf16_kernel<DD><<<gwq, AB_THREADS, lds_dq, stream>>>(gq_geom, qkv, o, dout, lse, lse2, delta, dqkv, part_q, pq, T, sc, sl2); \
      DH_LAUNCH_CHECK();                                                                                                       \
      attn_bwd_dkv_bf16_kernel<DD><<<gwk, AB_THREADS, lds_dkv, stream>>>(gk_geom, qkv, dout, lse2, delta, part_kv, pk, T, sc, sl2); \
    }                                                                                                                          \
    DH_LAUNCH_CHECK();                                                                                                         \
    if (nb_q + nb_k > 0) {                                                                                                     \
      attn_bwd_reduce_kernel<DD><<<nb_q + nb_k, 256, 0, stream>>>(part_q, dqkv, pq, lay.ch_q, sc, nb_q, gq.x, gq.y, part_kv, gk_geom, pk, \
                                                                 gk.x, gk.y);                                                  \
      DH_LAUNCH_CHECK();                                                                                                       \
    }                                                                                                                          \
  } while (0)
  if (d == 128) DH_ATTN_BWD(128, 0); else DH_ATTN_BWD(64, 1);
#undef DH_ATTN_BWD
  return DH_OK;
}
