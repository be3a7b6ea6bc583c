// float32 causal grouped-query attention, forward and backward, for the fp32 configuration, on the float32 matrix
// instruction (v_mfma_f32_16x16x4_f32: float32 operands, products and sums).
// Layout: qkv[T, (nq+2nkv)*d] = [q heads | k heads | v heads], o[T, nq*d], lse[nq, T],
// delta[nq, T]; tokens are sequence-major and attention never crosses a sequence boundary.
// Keys and values come from kv[batch*(q_off+seq), ldkv] = [k heads | v heads] per row: the packed qkv rows
// themselves for plain attention (q_off = 0), or a gathered buffer whose first q_off rows per sequence belong to
// earlier context-parallel ranks; query i of a sequence sits at position q_off + i.  dK/dV go to dkv likewise.
//
// Bound: latency -- a head of this configuration has a few hundred rows.  A block owns 16 rows (queries for the forward and
// dQ kernels, keys for dK/dV) of one head; its eight or four waves take the 16-row tiles of the other side in turn and meet in LDS
// at the end, in wave order (no atomics: results do not depend on scheduling).  Operands go from memory (L1/L2) straight
// into fragments.  Score tiles are formed transposed where that keeps a row's statistics in its lane, and a tile of
// probabilities feeds the next product from the registers it was formed in: the instruction's k index of lane group g and
// step e may be any row as long as both operands agree, and row 4g + e is the one the lane already holds.
// 128 tokens, 4 heads of 64: forward 26 -> 7 us, backward 62 -> 19 us against one wave per row with dot products.  Looking for
// infinities and NaNs in the tiles that have masked entries costs nothing there (1024 tokens, 4 heads of 64: backward 172.8 ->
// 173.6 us), 2-4 % with heads of 128 and, at 300 tokens, 11 % with heads of 256, whose elements are fetched twice for it.
#include <algorithm>
#include <type_traits>
#include "common.h"

// Waves of a block: eight where the fragments of a 64-wide head leave room for two waves per SIMD, else four.
template <int DT> constexpr int a32_waves() { return DT <= 4 ? 8 : 4; }
#define A32_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0)

// Row fragments: lane (l16, g) holds elements 16c + 4g + e of row l16 (c < DT chunks of 16, zero beyond d).
template <int DT>
struct RowFrag {
  float v[DT][4];
  __device__ __forceinline__ void load(const float* __restrict__ row, bool valid, int g, int d) {
#pragma unroll
    for (int c = 0; c < DT; c++) {
      const int k = 16 * c + 4 * g;
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
      if (valid && k < d) x = *reinterpret_cast<const float4*>(row + k);  // d is a multiple of 4
      v[c][0] = x.x; v[c][1] = x.y; v[c][2] = x.z; v[c][3] = x.w;
    }
  }
};
// 16x16 tile of dot products: result rows = rows of a, columns (lane l16) = rows of b.
template <int DT>
__device__ __forceinline__ f32x4 dot_tile(const RowFrag<DT>& a, const RowFrag<DT>& b) {
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
  for (int c = 0; c < DT; c++) {  // two chains, so that a product does not wait for the one before it
    s0 = A32_MFMA(a.v[c][0], b.v[c][0], s0);
    s1 = A32_MFMA(a.v[c][1], b.v[c][1], s1);
    s0 = A32_MFMA(a.v[c][2], b.v[c][2], s0);
    s1 = A32_MFMA(a.v[c][3], b.v[c][3], s1);
  }
  return s0 + s1;
}
// acc[c] (rows = elements 16c.. of the head, column l16) += rows[4g+e][16c + l16] * p[e], summed over the 16 rows.  The
// elements can be fetched ahead (EARLY: heads up to 128, where they fit the registers), together with the row fragments.
template <int DT>
struct ColFrag {
  static constexpr bool EARLY = DT <= 8;
  const float* base;
  size_t ld;
  float x[EARLY ? DT : 1][4];
  int row0, row_last, l16, g, d;
  __device__ __forceinline__ const float* row(int j) const { return base + (size_t)min(row0 + j, row_last) * ld; }  // p is zero where clamped
  __device__ __forceinline__ void start(const float* __restrict__ base_, size_t ld_, int row0_, int row_last_, int l16_, int g_, int d_) {
    base = base_; ld = ld_; row0 = row0_; row_last = row_last_; l16 = l16_; g = g_; d = d_;
    if constexpr (EARLY) {
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int c = 0; c < DT; c++) x[c][e] = 16 * c + l16 < d ? row(4 * g + e)[16 * c + l16] : 0.f;
    }
  }
  __device__ __forceinline__ float elem(int c, int e) const {
    if constexpr (EARLY) return x[c][e];
    else return 16 * c + l16 < d ? row(4 * g + e)[16 * c + l16] : 0.f;
  }
  __device__ __forceinline__ void accumulate(f32x4 (&acc)[DT], const f32x4 p) const {
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int c = 0; c < DT; c++) acc[c] = A32_MFMA(elem(c, e), p[e], acc[c]);
  }
  // Largest magnitude among the elements this lane holds, as an integer that orders infinities and NaNs last.
  __device__ __forceinline__ unsigned largest() const {
    unsigned t = 0;
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int c = 0; c < DT; c++) t = max(t, __float_as_uint(elem(c, e)) & 0x7fffffffu);
    return t;
  }
  // The same sum for a tile in which some rows do not count for some columns (partial; bit e of seen: row 4g+e counts for
  // column l16; p is zero where it does not).  The instruction multiplies those rows too, and zero times an infinity or a
  // NaN is a NaN: such a tile is summed over the rows that count alone if its elements are not all finite.
  template <typename Partial>
  __device__ __forceinline__ void accumulate_seen(f32x4 (&acc)[DT], const f32x4 p, Partial partial, int seen) const {
    if (!partial || __all(largest() < 0x7f800000u)) {
      accumulate(acc, p);
      return;
    }
#pragma unroll 1
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float pj = __shfl(p[e], 16 * q + l16, 64);
        const bool counts = (__shfl(seen, 16 * q + l16, 64) >> e) & 1;
        const float* r = row(4 * q + e) + 4 * g;
        if (counts) {
#pragma unroll
          for (int c = 0; c < DT; c++)
            if (16 * c + 4 * g < d) {
              const f32x4 x4 = *reinterpret_cast<const f32x4*>(r + 16 * c);
#pragma unroll
              for (int i = 0; i < 4; i++) acc[c][i] = fmaf(x4[i], pj, acc[c][i]);
            }
        }
      }
  }
};
__device__ __forceinline__ float group_sum(float v) {  // over the four lane groups of a column
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}

// Runs a tile's body for a partial tile (true) or a whole one.  Two copies of the body, so that whole tiles carry nothing of the
// masks; one with a run-time switch where the fragments leave no registers for two (heads above 128).
template <int DT, typename Fn>
__device__ __forceinline__ void with_partial(bool partial, Fn body) {
  partial = __builtin_amdgcn_readfirstlane(partial);
  if constexpr (DT > 8) body(partial);
  else if (partial) body(std::true_type{});
  else body(std::false_type{});
}

// grid (16-query tiles per sequence, nq, sequences)
template <int DT>
__global__ __launch_bounds__(64 * a32_waves<DT>()) void attn_fwd_f32_kernel(int seq, int nq, int nkv, int d, const float* __restrict__ qkv,
                                                                      const float* __restrict__ kv, int ldkv, int q_off,
                                                                      float* __restrict__ o, float* __restrict__ lse, int T) {
  constexpr int A32_WAVES = a32_waves<DT>();
  __shared__ float ms[A32_WAVES][16], ls[A32_WAVES][16];
  extern __shared__ float os[];  // [16 queries][DT*16 + 4]
  constexpr int LD = DT * 16 + 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z, hk = h / (nq / nkv), i0 = (gridDim.x - 1 - blockIdx.x) * 16, iq = i0 + l16;  // longest rows first
  const int ld = (nq + 2 * nkv) * d;
  const float scale = 1.0f / sqrtf((float)d);
  const size_t tok = (size_t)b * seq + min(iq, seq - 1);
  RowFrag<DT> q;
  q.load(qkv + tok * ld + (size_t)h * d, iq < seq, g, d);
#pragma unroll
  for (int c = 0; c < DT; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) q.v[c][e] *= scale;
  const float* kbase = kv + (size_t)b * (q_off + seq) * ldkv + (size_t)hk * d;
  const float* vbase = kbase + (size_t)nkv * d;
  const int key_last = q_off + seq - 1, last = min(q_off + iq, key_last), tiles = (q_off + min(i0 + 16, seq) + 15) / 16;
  float m = -INFINITY, l = 0.f;
  f32x4 acc[DT];
#pragma unroll
  for (int c = 0; c < DT; c++) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto tile = [&](auto partial, int j0) {  // partial: some keys of the tile lie behind some of the queries
    RowFrag<DT> k;
    k.load(kbase + (size_t)min(j0 + l16, key_last) * ldkv, true, g, d);
    ColFrag<DT> vc;
    vc.start(vbase, ldkv, j0, key_last, l16, g, d);
    f32x4 s = dot_tile<DT>(k, q);  // rows = keys, column = query
    int seen = 0;
    if (partial) {
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if (j0 + 4 * g + e > last) s[e] = -INFINITY;
        else seen |= 1 << e;
      }
    }
    const float mn = fmaxf(m, group_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
    if (__any(mn > m)) {
      const float alpha = mn == -INFINITY ? 1.f : expf(m - mn);  // a row past the sequence end of a masked tile sees no key
      l *= alpha;
#pragma unroll
      for (int c = 0; c < DT; c++) acc[c] *= alpha;
      m = mn;
    }
    f32x4 p;
#pragma unroll
    for (int e = 0; e < 4; e++) p[e] = s[e] == -INFINITY ? 0.f : expf(s[e] - m);
    l += group_sum(p[0] + p[1] + p[2] + p[3]);
    vc.accumulate_seen(acc, p, partial, seen);
  };
  for (int t = wave; t < tiles; t += A32_WAVES) {
    with_partial<DT>(t * 16 + 15 > q_off + i0, [&](auto partial) { tile(partial, t * 16); });
  }
  if (g == 0) { ms[wave][l16] = m; ls[wave][l16] = l; }
  __syncthreads();
  float M = ms[0][l16], L = 0.f;
#pragma unroll
  for (int w = 1; w < A32_WAVES; w++) M = fmaxf(M, ms[w][l16]);
#pragma unroll
  for (int w = 0; w < A32_WAVES; w++) L += ls[w][l16] == 0.f ? 0.f : ls[w][l16] * expf(ms[w][l16] - M);
  if (M == -INFINITY) L = NAN;  // every score the row sees is minus infinity (or a NaN): no softmax
  const float f = l == 0.f && L == L ? 0.f : expf(m - M) / L;
  for (int w = 0; w < A32_WAVES; w++) {  // the waves' shares, added in wave order
    if (wave == w) {
#pragma unroll
      for (int c = 0; c < DT; c++) {
        f32x4* dst = reinterpret_cast<f32x4*>(os + l16 * LD + 16 * c + 4 * g);
        const f32x4 v = acc[c] * f;
        *dst = w == 0 ? v : *dst + v;
      }
    }
    __syncthreads();
  }
  for (int x = threadIdx.x; x < 16 * (d / 4); x += blockDim.x) {
    const int r = x / (d / 4), c4 = (x % (d / 4)) * 4;
    if (i0 + r < seq)
      *reinterpret_cast<f32x4*>(o + ((size_t)b * seq + i0 + r) * nq * d + (size_t)h * d + c4) = *reinterpret_cast<const f32x4*>(os + r * LD + c4);
  }
  if (wave == 0 && g == 0 && iq < seq) lse[(size_t)h * T + tok] = M + logf(L);
}

struct A32Bwd {
  int seq, nq, nkv, d, ldkv, q_off, lddkv, T;
  const float *qkv, *kv, *o, *dout, *lse;
  float *delta, *dqkv, *dkv;
};
// sum_c dout[c] * o[c] of the row the lane's fragments hold a part of
template <int DT>
__device__ __forceinline__ float row_delta(const RowFrag<DT>& dof, const float* o, bool valid, int g, int d) {
  RowFrag<DT> of;
  of.load(o, valid, g, d);
  float dl = 0.f;
#pragma unroll
  for (int c = 0; c < DT; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) dl = fmaf(dof.v[c][e], of.v[c][e], dl);
  return group_sum(dl);
}

// dQ of query tile `tile_q` of head h, sequence b; also stores delta[h, t] = sum_c dout[t,h,c] * o[t,h,c].
template <int DT>
__device__ __forceinline__ void attn_bwd_dq_f32(const A32Bwd& a, int tile_q, int h, int b, float* os) {
  constexpr int A32_WAVES = a32_waves<DT>();
  const int seq = a.seq, nq = a.nq, nkv = a.nkv, d = a.d, ldkv = a.ldkv, q_off = a.q_off, T = a.T;
  const float *__restrict__ qkv = a.qkv, *__restrict__ kv = a.kv, *__restrict__ o = a.o, *__restrict__ dout = a.dout, *__restrict__ lse = a.lse;
  float *__restrict__ delta = a.delta, *__restrict__ dqkv = a.dqkv;
  constexpr int LD = DT * 16 + 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
  const int hk = h / (nq / nkv), i0 = tile_q * 16, iq = i0 + l16;
  const int ld = (nq + 2 * nkv) * d;
  const float scale = 1.0f / sqrtf((float)d);
  const size_t tok = (size_t)b * seq + min(iq, seq - 1);
  RowFrag<DT> q, dof;
  dof.load(dout + tok * nq * d + (size_t)h * d, iq < seq, g, d);
  const float dl = row_delta<DT>(dof, o + tok * nq * d + (size_t)h * d, iq < seq, g, d);
  if (wave == 0 && g == 0 && iq < seq) delta[(size_t)h * T + tok] = dl;
  q.load(qkv + tok * ld + (size_t)h * d, iq < seq, g, d);
#pragma unroll
  for (int c = 0; c < DT; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) q.v[c][e] *= scale;
  const float Lq = lse[(size_t)h * T + tok];
  const float* kbase = kv + (size_t)b * (q_off + seq) * ldkv + (size_t)hk * d;
  const float* vbase = kbase + (size_t)nkv * d;
  const int key_last = q_off + seq - 1, last = min(q_off + iq, key_last), tiles = (q_off + min(i0 + 16, seq) + 15) / 16;
  f32x4 acc[DT];
#pragma unroll
  for (int c = 0; c < DT; c++) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto tile = [&](auto partial, int j0) {
    const size_t row = (size_t)min(j0 + l16, key_last) * ldkv;
    RowFrag<DT> k, v;
    k.load(kbase + row, true, g, d);
    v.load(vbase + row, true, g, d);
    ColFrag<DT> kc;
    kc.start(kbase, ldkv, j0, key_last, l16, g, d);
    const f32x4 s = dot_tile<DT>(k, q);
    const f32x4 dp = dot_tile<DT>(v, dof);
    f32x4 ds;
    int seen = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const bool counts = !partial || j0 + 4 * g + e <= last;
      ds[e] = counts ? expf(s[e] - Lq) * (dp[e] - dl) : 0.f;
      seen |= counts ? 1 << e : 0;
    }
    kc.accumulate_seen(acc, ds, partial, seen);
  };
  for (int t = wave; t < tiles; t += A32_WAVES) {
    with_partial<DT>(t * 16 + 15 > q_off + i0, [&](auto partial) { tile(partial, t * 16); });
  }
  for (int w = 0; w < A32_WAVES; w++) {
    if (wave == w) {
#pragma unroll
      for (int c = 0; c < DT; c++) {
        f32x4* dst = reinterpret_cast<f32x4*>(os + l16 * LD + 16 * c + 4 * g);
        *dst = w == 0 ? acc[c] : *dst + acc[c];
      }
    }
    __syncthreads();
  }
  for (int x = threadIdx.x; x < 16 * (d / 4); x += blockDim.x) {
    const int r = x / (d / 4), c4 = (x % (d / 4)) * 4;
    if (i0 + r < seq)
      *reinterpret_cast<f32x4*>(dqkv + ((size_t)b * seq + i0 + r) * ld + (size_t)h * d + c4) =
          *reinterpret_cast<const f32x4*>(os + r * LD + c4) * scale;
  }
}

// dK, dV of key tile `tile_k` of key/value head hk, sequence b: every (query head of the group, query tile) pair.  OWN_DELTA: delta is formed here as the dQ tiles do,
// which may not have stored it yet.
template <int DT, bool OWN_DELTA>
__device__ __forceinline__ void attn_bwd_dkv_f32(const A32Bwd& a, int tile_k, int hk, int b, float* os) {  // os: [16 keys][dK | dV], row pitch 2*DT*16 + 4
  constexpr int A32_WAVES = a32_waves<DT>();
  const int seq = a.seq, nq = a.nq, nkv = a.nkv, d = a.d, ldkv = a.ldkv, q_off = a.q_off, T = a.T, lddkv = a.lddkv;
  const float *__restrict__ qkv = a.qkv, *__restrict__ kv = a.kv, *__restrict__ dout = a.dout, *__restrict__ lse = a.lse, *__restrict__ delta = a.delta;
  float* __restrict__ dkv = a.dkv;
  constexpr int LD = 2 * DT * 16 + 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
  const int grp = nq / nkv, S = q_off + seq, j0 = tile_k * 16, jk = j0 + l16;
  const int ld = (nq + 2 * nkv) * d;
  const float scale = 1.0f / sqrtf((float)d);
  const float* krow = kv + ((size_t)b * S + min(jk, S - 1)) * ldkv + (size_t)hk * d;
  RowFrag<DT> k, v;
  k.load(krow, jk < S, g, d);
  v.load(krow + (size_t)nkv * d, jk < S, g, d);
#pragma unroll
  for (int c = 0; c < DT; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) k.v[c][e] *= scale;
  f32x4 dk[DT], dv[DT];
#pragma unroll
  for (int c = 0; c < DT; c++) dk[c] = dv[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int t_first = max(j0 - q_off, 0) / 16, tiles = (seq + 15) / 16 - t_first;  // query tiles that see any key of this one
  auto tile = [&](auto partial, int h, int i0) {  // partial: some queries of the tile lie before some of the keys, or past the end
    const size_t tok0 = (size_t)b * seq, row = tok0 + min(i0 + l16, seq - 1);
    const float* qb = qkv + tok0 * ld + (size_t)h * d;
    const float* ob = dout + tok0 * nq * d + (size_t)h * d;
    RowFrag<DT> q, dof;
    q.load(qkv + row * ld + (size_t)h * d, true, g, d);
    dof.load(dout + row * nq * d + (size_t)h * d, true, g, d);
    ColFrag<DT> qc, oc;
    oc.start(ob, (size_t)nq * d, i0, seq - 1, l16, g, d);
    qc.start(qb, ld, i0, seq - 1, l16, g, d);
    float own = 0.f;
    if constexpr (OWN_DELTA) own = row_delta<DT>(dof, a.o + row * nq * d + (size_t)h * d, true, g, d);
    const f32x4 s = dot_tile<DT>(q, k);  // rows = queries, column = key
    const f32x4 dp = dot_tile<DT>(dof, v);
    f32x4 p, ds;
    int seen = 0;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int i = i0 + 4 * g + e;
      const size_t st = (size_t)h * T + tok0 + min(i, seq - 1);
      const bool counts = !partial || (i < seq && q_off + i >= jk);
      p[e] = counts ? expf(s[e] - lse[st]) : 0.f;
      const float dl = OWN_DELTA ? __shfl(own, 4 * g + e, 64) : delta[st];  // lane l16 holds row i0 + l16's
      ds[e] = counts ? p[e] * (dp[e] - dl) : 0.f;
      seen |= counts ? 1 << e : 0;
    }
    oc.accumulate_seen(dv, p, partial, seen);
    qc.accumulate_seen(dk, ds, partial, seen);
  };
  for (int x = wave; x < grp * tiles; x += A32_WAVES) {
    const int h = hk * grp + x / tiles, i0 = (t_first + x % tiles) * 16;
    with_partial<DT>(i0 + 16 > seq || q_off + i0 < j0 + 15, [&](auto partial) { tile(partial, h, i0); });
  }
  for (int w = 0; w < A32_WAVES; w++) {
    if (wave == w) {
#pragma unroll
      for (int c = 0; c < DT; c++) {
        f32x4* dst = reinterpret_cast<f32x4*>(os + l16 * LD + 16 * c + 4 * g);
        f32x4* dst2 = reinterpret_cast<f32x4*>(os + l16 * LD + DT * 16 + 16 * c + 4 * g);
        *dst = w == 0 ? dk[c] : *dst + dk[c];
        *dst2 = w == 0 ? dv[c] : *dst2 + dv[c];
      }
    }
    __syncthreads();
  }
  for (int x = threadIdx.x; x < 16 * (d / 4); x += blockDim.x) {
    const int r = x / (d / 4), c4 = (x % (d / 4)) * 4;
    if (j0 + r >= S) continue;
    float* dst = dkv + ((size_t)b * S + j0 + r) * lddkv + (size_t)hk * d + c4;
    *reinterpret_cast<f32x4*>(dst) = *reinterpret_cast<const f32x4*>(os + r * LD + c4) * scale;
    *reinterpret_cast<f32x4*>(dst + (size_t)nkv * d) = *reinterpret_cast<const f32x4*>(os + r * LD + DT * 16 + c4);
  }
}

// The two as launches of their own, grids (16-query tiles, longest rows first, nq, sequences) and (16-key tiles, nkv, sequences) ...
template <int DT>
__global__ __launch_bounds__(64 * a32_waves<DT>()) void attn_bwd_dq_f32_kernel(const A32Bwd a) {
  extern __shared__ float os[];
  attn_bwd_dq_f32<DT>(a, gridDim.x - 1 - blockIdx.x, blockIdx.y, blockIdx.z, os);
}
template <int DT>
__global__ __launch_bounds__(64 * a32_waves<DT>()) void attn_bwd_dkv_f32_kernel(const A32Bwd a) {
  extern __shared__ float os[];
  attn_bwd_dkv_f32<DT, false>(a, blockIdx.x, blockIdx.y, blockIdx.z, os);
}
// ... and as one, grid (key tiles * nkv + query tiles * nq, 1, sequences).
template <int DT>
__global__ __launch_bounds__(64 * a32_waves<DT>()) void attn_bwd_f32_kernel(const A32Bwd a, int tiles_k, int tiles_q) {
  extern __shared__ float os[];
  const int x = blockIdx.x, n_k = tiles_k * a.nkv;
  if (x < n_k) attn_bwd_dkv_f32<DT, true>(a, x % tiles_k, x / tiles_k, blockIdx.z, os);
  else attn_bwd_dq_f32<DT>(a, tiles_q - 1 - (x - n_k) % tiles_q, (x - n_k) / tiles_q, blockIdx.z, os);
}

static int check_f32(int d) {
  if (d > 256 || d % 4) DH_FAIL(DH_ERR_SHAPE, "attention (fp32): head_dim %d must be a multiple of 4, at most 256", d);
  return DH_OK;
}

// Sequences of one launch: the third dimension of a grid holds 65535 blocks.
#define A32_MAX_BATCH 65535
#define A32_ONE_LAUNCH 2048  // blocks of a backward pass in one launch (see bwd_f32)

template <int DT>
static int fwd_f32(int batch, int seq, int nq, int nkv, int d, const float* qkv, const float* kv, int ldkv, int q_off, float* o, float* lse,
                   hipStream_t stream) {
  const size_t ld = (size_t)(nq + 2 * nkv) * d;
  for (int b0 = 0; b0 < batch; b0 += A32_MAX_BATCH) {
    const size_t t0 = (size_t)b0 * seq, k0 = (size_t)b0 * (q_off + seq);
    attn_fwd_f32_kernel<DT><<<dim3((seq + 15) / 16, nq, std::min(batch - b0, A32_MAX_BATCH)), 64 * a32_waves<DT>(), 16 * (DT * 16 + 4) * sizeof(float), stream>>>(
        seq, nq, nkv, d, qkv + t0 * ld, kv + k0 * ldkv, ldkv, q_off, o + t0 * nq * d, lse + t0, batch * seq);
    DH_LAUNCH_CHECK();
  }
  return DH_OK;
}

int dh_launch_attn_fwd_f32(int batch, int seq, int nq, int nkv, int d, const float* qkv, const float* kv, int ldkv,
                           int q_off, float* o, float* lse, hipStream_t stream) {
  int rc = check_f32(d);
  if (rc) return rc;
  if (batch * seq == 0) return DH_OK;
  if (!kv) { kv = qkv + (size_t)nq * d; ldkv = (nq + 2 * nkv) * d; q_off = 0; }
  if (d <= 32) return fwd_f32<2>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, lse, stream);
  if (d <= 64) return fwd_f32<4>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, lse, stream);
  if (d <= 128) return fwd_f32<8>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, lse, stream);
  return fwd_f32<16>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, lse, stream);
}

template <int DT>
static int bwd_f32(int batch, int seq, int nq, int nkv, int d, const float* qkv, const float* kv, int ldkv, int q_off, const float* o,
                   const float* dout, const float* lse, float* dqkv, float* dkv, int lddkv, float* delta, hipStream_t stream) {
  const int T = batch * seq;
  const size_t ld = (size_t)(nq + 2 * nkv) * d;
  for (int b0 = 0; b0 < batch; b0 += A32_MAX_BATCH) {
    const size_t t0 = (size_t)b0 * seq, k0 = (size_t)b0 * (q_off + seq);
    const int nb = std::min(batch - b0, A32_MAX_BATCH);
    const A32Bwd a = {seq, nq, nkv, d, ldkv, q_off, lddkv, T, qkv + t0 * ld, kv + k0 * ldkv, o + t0 * nq * d, dout + t0 * nq * d, lse + t0,
                      delta + t0, dqkv + t0 * ld, dkv + k0 * lddkv};
    const int tiles_q = (seq + 15) / 16, tiles_k = (q_off + seq + 15) / 16;
    const size_t lds_q = 16 * (DT * 16 + 4) * sizeof(float), lds_k = 16 * (2 * DT * 16 + 4) * sizeof(float);
    // A few rounds of blocks are chains of latencies, and one launch makes the two kinds' chains run side by side (us, two launches and one: 4 heads x 128 of 64
    // 19.2 and 10.2, 8:1 x 128 of 128 99.7 and 87, 8 x 1000 of 64 132 and 110, 16 x 1024 of 64, 2048 blocks, 244 and 226; the same bits).  Further rounds fill the units by
    // themselves, and the sums for delta that every key tile makes again are work there.
    if constexpr (DT <= 8) {
      if (((long long)tiles_q * nq + (long long)tiles_k * nkv) * nb <= A32_ONE_LAUNCH) {
        attn_bwd_f32_kernel<DT><<<dim3(tiles_q * nq + tiles_k * nkv, 1, nb), 64 * a32_waves<DT>(), lds_k, stream>>>(a, tiles_k, tiles_q);
        DH_LAUNCH_CHECK();
        continue;
      }
    }
    attn_bwd_dq_f32_kernel<DT><<<dim3(tiles_q, nq, nb), 64 * a32_waves<DT>(), lds_q, stream>>>(a);
    DH_LAUNCH_CHECK();
    attn_bwd_dkv_f32_kernel<DT><<<dim3(tiles_k, nkv, nb), 64 * a32_waves<DT>(), lds_k, stream>>>(a);
    DH_LAUNCH_CHECK();
  }
  return DH_OK;
}

int dh_launch_attn_bwd_f32(int batch, int seq, int nq, int nkv, int d, const float* qkv, const float* kv, int ldkv,
                           int q_off, const float* o, const float* dout, const float* lse, float* dqkv, float* dkv, int lddkv,
                           float* delta, hipStream_t stream) {
  int rc = check_f32(d);
  if (rc) return rc;
  if (batch * seq == 0) return DH_OK;
  if (!kv) {
    kv = qkv + (size_t)nq * d; dkv = dqkv + (size_t)nq * d;
    ldkv = lddkv = (nq + 2 * nkv) * d; q_off = 0;
  }
  if (d <= 32) return bwd_f32<2>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, dout, lse, dqkv, dkv, lddkv, delta, stream);
  if (d <= 64) return bwd_f32<4>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, dout, lse, dqkv, dkv, lddkv, delta, stream);
  if (d <= 128) return bwd_f32<8>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, dout, lse, dqkv, dkv, lddkv, delta, stream);
  return bwd_f32<16>(batch, seq, nq, nkv, d, qkv, kv, ldkv, q_off, o, dout, lse, dqkv, dkv, lddkv, delta, stream);
}
