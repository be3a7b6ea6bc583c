// Row-wise and element-wise operators of the layer: RMSNorm (with the residual add of the
// bias-dropout-add operator fused in, dropout p = 0), RoPE, SwiGLU, residual add.
// All are HBM-bound: every tensor is read or written exactly once with 16-byte (bf16) or
// 2x16-byte (fp32) accesses per thread; reductions are wave/block reductions in registers.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include "common.h"

#define ROW_THREADS 256

// ------------------------------------------------------------------------------------ operand that a collective delivers
// A row operand read as it is (SUM = false) or as the sum of the collective's partial buffers (SUM = true): added in rank
// order in float32 and rounded to the storage type, the bits the stand-in kernel would have stored.  The operator behind a
// reduction then reads the partials itself: one pass over the reduced tensor less on each side and one launch less.
template <typename T, bool SUM> struct RowSrc;
template <typename T> struct RowSrc<T, false> {
  const T* p;
  __device__ __forceinline__ bool present() const { return p != nullptr; }
  template <bool AHEAD = true> __device__ __forceinline__ void load(Vec8<T>& v, size_t off) const { v.load(p + off); }
};
template <typename T> struct RowSrc<T, true> {
  PartPtrs parts;
  int n;
  __device__ __forceinline__ bool present() const { return true; }
  // AHEAD: seven loads in flight (eight ranks: all of them), or three (four ranks); else one after the other.  The two counts are apart for the
  // compiler's sake: with the three behind the loop over seven it waited for each of the first four.
  template <bool AHEAD = true> __device__ __forceinline__ void load(Vec8<T>& v, size_t off) const {
    v.load_stream((const T*)parts.p[0] + off);
    int r = 1;
    auto take = [&](auto count) {
      constexpr int N = decltype(count)::value;
      Vec8<T> w[N];
#pragma unroll
      for (int u = 0; u < N; u++) w[u].load_stream((const T*)parts.p[r + u] + off);
#pragma unroll
      for (int u = 0; u < N; u++)
#pragma unroll
        for (int i = 0; i < 8; i++) v.v[i] += w[u].v[i];
      r += N;
    };
    if (AHEAD && n >= 8) {
      while (r + 7 <= n) take(std::integral_constant<int, 7>());
    } else if (AHEAD) {
      while (r + 3 <= n) take(std::integral_constant<int, 3>());
    }
    while (r < n) take(std::integral_constant<int, 1>());
#pragma unroll
    for (int i = 0; i < 8; i++) v.v[i] = to_f32(from_f32<T>(v.v[i]));
  }
};

// ------------------------------------------------------------------------------------ RMSNorm fwd
// One 256-thread block per row.  Thread t owns columns (t + 256*c)*8 .. +7 for c < NCH and keeps
// them in registers between the sum-of-squares pass and the scale pass.
template <typename T, int NCH, bool SUM>
__global__ __launch_bounds__(ROW_THREADS) void rmsnorm_fwd_kernel(const T* __restrict__ x, const RowSrc<T, SUM> res,
                                                                  const T* __restrict__ gamma, float eps,
                                                                  T* __restrict__ x_out, T* __restrict__ h,
                                                                  float* __restrict__ rstd, int H) {
  __shared__ float red[8];
  const size_t row = blockIdx.x;
  const T* xr = x + row * H;
  Vec8<T> v[NCH];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (threadIdx.x + ROW_THREADS * c) * 8;
    if (col < H) {
      v[c].load(xr + col);
      if (res.present()) {
        Vec8<T> r;
        res.load(r, row * H + col);
#pragma unroll
        for (int i = 0; i < 8; i++) v[c].v[i] = to_f32(from_f32<T>(v[c].v[i] + r.v[i]));
        v[c].store(x_out + row * H + col);
      }
#pragma unroll
      for (int i = 0; i < 8; i++) ss += v[c].v[i] * v[c].v[i];
    }
  }
  ss = block256_sum(ss, red);
  float r = 1.0f / sqrtf(ss / (float)H + eps);
  if (threadIdx.x == 0) rstd[row] = r;
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (threadIdx.x + ROW_THREADS * c) * 8;
    if (col < H) {
      Vec8<T> g;
      g.load(gamma + col);
#pragma unroll
      for (int i = 0; i < 8; i++) g.v[i] = g.v[i] * v[c].v[i] * r;
      g.store(h + row * H + col);
    }
  }
}

// ------------------------------------------------------------------------------------ RMSNorm bwd
// Block b handles rows [b*RPB, (b+1)*RPB).  dx = rstd*(gh - xh*mean(gh*xh)) (+ dres), gh = gamma*dy,
// xh = x*rstd.  The next row is already in flight while the current one is reduced.  The gain
// gradient sum_t dy*xh is accumulated per thread over the block's rows and written as one partial
// row per block; colsum_finish_kernel then adds the partial rows in an order fixed by the shapes, so the result
// does not depend on scheduling.
// Rows a backward-norm block walks (its partial gain gradient is one row of the column-sum input): 8, fewer for
// short inputs so that a couple of hundred blocks exist.
__host__ __device__ static inline int norm_bwd_rpb(int rows) { return rows >= 4096 ? 8 : rows >= 1024 ? 4 : rows >= 512 ? 2 : 1; }
// Short rows leave threads of a block idle (1024 columns are 128 threads' work), and its rows are a chain of loads and sums one after the other: G
// groups of threads take every G-th row each, side by side.  Columns, and the order of a row's sum, are those of one group.
// us of the bare operator with the column sums behind it, one group and four, bf16: RMSNorm, 2048 x 512 8.3 -> 6.9, 8192 x 512 14.1 -> 12.6, LayerNorm 10.3 -> 7.4, 17.3 ->
// 14.3 (float32 8.8 -> 8.4 and 15.7 -> 16.4, 10.5 -> 9.6 and 17.9 -> 17.4).  One and two: RMSNorm, 1024 x 1024 7.8 -> 7.1, 2048 x 1024 9.6 -> 9.5, LayerNorm 9.7 -> 8.2, 11.9 ->
// 11.3, 2048 x 640 8.6 -> 7.8 and 10.6 -> 9.5.  Two groups are drawn by what they gain inside a layer, where the norm reads the ranks' partial buffers one after the other or what
// a product has just written: backward passes of small layers, bf16, 1024 to 8192 rows of 640 to 1024, 1.00 to 1.07 times as fast on one, two and eight ranks (4000 x
// 1024 1.00, 1.02, 1.01; 8192 x 1024 1.01, 1.04, 1.00), float32 up to 2048 rows 1.00 to 1.04, 4000 rows 0.99.  The bare operator in a loop gains less and loses beyond
// 4 MB a tensor (RMSNorm, bf16 4000 x 1024 12.8 -> 13.6, float32 2048 x 1024 10.6 -> 11.8).  The count does not ask where the gradient comes from: a reduction with its norm has the
// bits of the two apart.  LayerNorm beyond 2048 rows keeps one group (bare, 4000 x 1024 15.1 -> 16.3; in layers 1.00 to 1.05).  Below 1024 rows a block has one or two.
template <typename T>
static int norm_bwd_groups(int rows, int H, bool layernorm) {
  if (rows < 1024 || H > 1024) return 1;
  if (H <= 512) return 4;
  return rows <= 2048 || (sizeof(T) == 2 && !layernorm) ? 2 : 1;
}
template <int G>
__device__ __forceinline__ float rows_sum(float v, float* red) {  // over the threads of the caller's group
  if constexpr (G == 1) return block256_sum(v, red);
  v = wave_sum(v);
  if constexpr (G == 2) {
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[wave] = v;
    __syncthreads();
    v = red[wave & 2] + red[(wave & 2) + 1];
  }
  return v;
}
// The groups' column sums (8 a thread), added in group order, to the partial row.
template <int G>
__device__ __forceinline__ void store_column_sums(float (&d)[8], float* row, int col, int H) {
  if constexpr (G > 1) {
    __shared__ float all[G][ROW_THREADS / G][8];
    const int grp = threadIdx.x / (ROW_THREADS / G), t = threadIdx.x % (ROW_THREADS / G);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; i++) all[grp][t][i] = d[i];
    __syncthreads();
    if (grp != 0) return;
#pragma unroll
    for (int k = 1; k < G; k++)
#pragma unroll
      for (int i = 0; i < 8; i++) d[i] += all[k][t][i];
  }
  if (col < H) {
    float4* p = reinterpret_cast<float4*>(row + col);
    p[0] = make_float4(d[0], d[1], d[2], d[3]);
    p[1] = make_float4(d[4], d[5], d[6], d[7]);
  }
}
template <typename T, int NCH, bool SUM, int G>
__global__ __launch_bounds__(ROW_THREADS) void rmsnorm_bwd_kernel(const RowSrc<T, SUM> dy, const T* __restrict__ x,
                                                                  const T* __restrict__ gamma,
                                                                  const float* __restrict__ rstd,
                                                                  const T* __restrict__ dres, T* __restrict__ dx,
                                                                  float* __restrict__ dg_partial, int rows, int H) {
  static_assert(G == 1 || NCH == 1, "groups are for rows of few threads");
  __shared__ float red[8];
  const int t = threadIdx.x % (ROW_THREADS / G), grp = threadIdx.x / (ROW_THREADS / G);
  Vec8<T> g[NCH];
  float dg[NCH][8];
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (t + ROW_THREADS * c) * 8;
    if (col < H) g[c].load(gamma + col);
#pragma unroll
    for (int i = 0; i < 8; i++) dg[c][i] = 0.f;
  }
  const int rpb = norm_bwd_rpb(rows);
  const size_t row0 = (size_t)blockIdx.x * rpb;
  const int nrows = min(rpb, rows - (int)row0);
  Raw8<T> ndy[SUM ? 1 : NCH], nx[NCH], nres[NCH];  // the next row, as fetched (partials are fetched when their row comes up)
  auto fetch = [&](size_t row) {
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      int col = (t + ROW_THREADS * c) * 8;
      if (col < H) {
        if constexpr (!SUM) ndy[c].load(dy.p + row * H + col);
        nx[c].load(x + row * H + col);
        if (dres != nullptr) nres[c].load(dres + row * H + col);
      }
    }
  };
  fetch(row0 + min(grp, nrows - 1));
  for (int rr = 0; rr < nrows; rr += G) {
    const bool mine = G == 1 || rr + grp < nrows;  // groups without a row in the last turn make the one before again
    const size_t row = row0 + (G == 1 ? rr : min(rr + grp, nrows - 1));
    const float r = rstd[row];
    Vec8<T> gh[NCH], xh[NCH];
    Raw8<T> rs[NCH];
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      const int col = (t + ROW_THREADS * c) * 8;
      if constexpr (!SUM) gh[c].from(ndy[c]);
      else if (col < H) dy.load(gh[c], row * H + col);
      xh[c].from(nx[c]);
      rs[c] = nres[c];
    }
    if (rr + G < nrows) fetch(row0 + (G == 1 ? rr + 1 : min(rr + G + grp, nrows - 1)));
    float dot = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      int col = (t + ROW_THREADS * c) * 8;
      if (col < H) {
#pragma unroll
        for (int i = 0; i < 8; i++) {
          xh[c].v[i] *= r;
          if (mine) dg[c][i] += gh[c].v[i] * xh[c].v[i];
          gh[c].v[i] *= g[c].v[i];
          dot += gh[c].v[i] * xh[c].v[i];
        }
      }
    }
    dot = rows_sum<G>(dot, red) / (float)H;
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      int col = (t + ROW_THREADS * c) * 8;
      if (col < H && mine) {
        Vec8<T> o;
#pragma unroll
        for (int i = 0; i < 8; i++) o.v[i] = r * (gh[c].v[i] - xh[c].v[i] * dot);
        if (dres != nullptr) {
#pragma unroll
          for (int i = 0; i < 8; i++) o.v[i] += rs[c].get(i);
        }
        o.store(dx + row * H + col);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NCH; c++) store_column_sums<G>(dg[c], dg_partial + (size_t)blockIdx.x * H, (t + ROW_THREADS * c) * 8, H);
}

// dst[col] += sum over the nrows partial rows of partial[row][col], in an order fixed by the shapes alone: a block owns
// 32 columns, its 32 slices of threads each add a contiguous 32nd of the rows in ascending order (16 loads in
// flight), and slice 0 adds the slices' sums in slice order.  Columns [0, H0) go to dst0, columns [H0, ld) to dst1.
// Bound by the latency of a slice's chain of load rounds, since the columns make few blocks: with 8 slices 1000 rows of 1024
// columns took 8.4 us and 1024 of 4096 as long, now 4.6 and 5.7.
#define COLSUM_SLICES 32
#define COLSUM_THREADS (32 * COLSUM_SLICES)
__global__ __launch_bounds__(COLSUM_THREADS) void colsum_finish_kernel(const float* __restrict__ partial, int nrows, int ld,
                                                            float* __restrict__ dst0, int H0, float* __restrict__ dst1) {
  __shared__ float part[COLSUM_SLICES][32];
  const int c = threadIdx.x & 31, slice = threadIdx.x >> 5, col = blockIdx.x * 32 + c;
  const int per = (nrows + COLSUM_SLICES - 1) / COLSUM_SLICES, r0 = slice * per, r1 = min(nrows, r0 + per);
  float s = 0.f;
  if (col < ld) {
    for (int b0 = r0; b0 < r1; b0 += 16) {
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; i++) v[i] = b0 + i < r1 ? partial[(size_t)(b0 + i) * ld + col] : 0.f;
#pragma unroll
      for (int i = 0; i < 16; i++) s += v[i];
    }
  }
  part[slice][c] = s;
  __syncthreads();
  if (slice == 0 && col < ld) {
    float t = part[0][c];
#pragma unroll
    for (int k = 1; k < COLSUM_SLICES; k++) t += part[k][c];
    if (col < H0) dst0[col] += t;
    else dst1[col - H0] += t;
  }
}

// ------------------------------------------------------------------------------------ RoPE
// In place on heads stored side by side in a row of `row_stride` elements.  A thread rotates 8
// pairs (i, i + d/2).  Angles are formed in double so that position*theta keeps full fp32 accuracy
// at long sequences: theta of the thread's first pair by one double exp2, the next seven by multiplying with
// ratio = base^(-2/d); the angle is reduced to [-pi, pi] in double, and only sine and cosine of the reduced
// angle are taken in float (absolute error ~1e-7).
// ADJACENT: pair i is elements (2i, 2i+1): the thread's 8 pairs are 16 consecutive elements.
// HEADS: heads a thread rotates, with one set of angles.  Bound by forming angles, sines and cosines with one head a thread, by memory with four
// (4096 rows of 40 heads of 128 21.0 -> 13.4 us, 6.3 TB/s; 8192 of 9 11.2 -> 7.3, 4000 of 32 of 64 10.3 -> 6.5, 4096 of 5 5.1 -> 4.5), by one thread's chain where
// there are few (256 of 5 3.65 us, four heads a thread 3.85): four from 2^17 threads of one head on.  Adjacent pairs in float32 stay with one: a lane's 64
// consecutive bytes of each of four heads come in more pieces than the angles are worth (4764 rows of 30 heads of 128 31 us, 35.5 with four; 12 shapes 5-13 % slower).
template <typename T, bool ADJACENT, int HEADS>
__global__ __launch_bounds__(256) void rope_kernel(T* __restrict__ t, size_t row0, unsigned threads, int seq, int pos0, int n_heads, int d, int row_stride,
                                                   double log2_base, double ratio, int inverse) {
  const int half = d / 2;
  const unsigned idx = blockIdx.x * 256 + threadIdx.x, chunks = half / 8, groups = (n_heads + HEADS - 1) / HEADS;
  if (idx >= threads) return;
  const int c = idx % chunks, head0 = idx / chunks % groups * HEADS;
  const size_t row = row0 + idx / (chunks * groups);
  const int pos = pos0 + (int)(row % seq);
  T* pa = t + row * row_stride + (size_t)head0 * d + (ADJACENT ? c * 16 : c * 8);
  Raw8<T> ra[HEADS], rb[HEADS];
#pragma unroll
  for (int h = 0; h < HEADS; h++)
    if (head0 + h < n_heads) {
      ra[h].load(pa + h * d);
      rb[h].load(pa + h * d + (ADJACENT ? 8 : half));
    }
  float sn[8], co[8];
  double theta = exp2(-2.0 * (double)(c * 8) / (double)d * log2_base);
#pragma unroll
  for (int i = 0; i < 8; i++) {
    double ang = (double)pos * theta;
    ang -= 6.283185307179586476925 * rint(ang * 0.15915494309189533577);
    theta *= ratio;
    sincosf((float)ang, &sn[i], &co[i]);
    if (inverse) sn[i] = -sn[i];
  }
#pragma unroll
  for (int h = 0; h < HEADS; h++) {
    if (head0 + h >= n_heads) break;
    Vec8<T> a, b, oa, ob;
    a.from(ra[h]);
    b.from(rb[h]);
    if (ADJACENT) {  // de-interleave: a = first elements of the 8 pairs, b = second elements
      Vec8<T> lo = a, hi = b;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        a.v[i] = lo.v[2 * i]; b.v[i] = lo.v[2 * i + 1];
        a.v[4 + i] = hi.v[2 * i]; b.v[4 + i] = hi.v[2 * i + 1];
      }
    }
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const float s = sn[i];
      oa.v[i] = fmaf(a.v[i], co[i], -__fmul_rn(b.v[i], s));  // the same roundings whatever HEADS is
      ob.v[i] = fmaf(b.v[i], co[i], __fmul_rn(a.v[i], s));
    }
    if (ADJACENT) {
      Vec8<T> lo, hi;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        lo.v[2 * i] = oa.v[i]; lo.v[2 * i + 1] = ob.v[i];
        hi.v[2 * i] = oa.v[4 + i]; hi.v[2 * i + 1] = ob.v[4 + i];
      }
      oa = lo; ob = hi;
    }
    oa.store(pa + h * d);
    ob.store(pa + h * d + (ADJACENT ? 8 : half));
  }
}

// ------------------------------------------------------------------------------------ SwiGLU
template <typename T>
__global__ void swiglu_fwd_kernel(const T* __restrict__ gu, T* __restrict__ a, int rows, int F) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  int chunks = F / 8;
  if (idx >= (size_t)rows * chunks) return;
  size_t row = idx / chunks;
  int col = (int)(idx % chunks) * 8;
  Vec8<T> g, u, o;
  g.load(gu + row * 2 * F + col);
  u.load(gu + row * 2 * F + F + col);
#pragma unroll
  for (int i = 0; i < 8; i++) o.v[i] = swiglu_fwd_elem(g.v[i], u.v[i]);
  o.store(a + row * F + col);
}

template <typename T>
__global__ void swiglu_bwd_kernel(const T* __restrict__ gu, const T* __restrict__ da, T* __restrict__ dgu, int rows, int F) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  int chunks = F / 8;
  if (idx >= (size_t)rows * chunks) return;
  size_t row = idx / chunks;
  int col = (int)(idx % chunks) * 8;
  Vec8<T> g, u, d, og, ou;
  g.load(gu + row * 2 * F + col);
  u.load(gu + row * 2 * F + F + col);
  d.load(da + row * F + col);
#pragma unroll
  for (int i = 0; i < 8; i++) swiglu_bwd_elem(g.v[i], u.v[i], d.v[i], og.v[i], ou.v[i]);
  og.store(dgu + row * 2 * F + col);
  ou.store(dgu + row * 2 * F + F + col);
}

// ------------------------------------------------------------------------------------ residual add
template <typename T, bool SUM, bool AHEAD = true>
__global__ void add_kernel(const T* __restrict__ a, const RowSrc<T, SUM> b, T* __restrict__ out, size_t n8) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n8) return;
  Vec8<T> x, y;
  x.load(a + idx * 8);
  b.template load<AHEAD>(y, idx * 8);
#pragma unroll
  for (int i = 0; i < 8; i++) x.v[i] += y.v[i];
  x.store(out + idx * 8);
}

// ------------------------------------------------------------------------------------ host side
static int nch_for(int H) {
  int n = (H + ROW_THREADS * 8 - 1) / (ROW_THREADS * 8);
  return n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : n <= 8 ? 8 : 0;
}

// Switch over the vectors a thread holds of a row; GO(N) launches.
#define NCH_SWITCH(name, H)                                                              \
  switch (nch_for(H)) {                                                                  \
    case 1: GO(1); break;                                                                \
    case 2: GO(2); break;                                                                \
    case 4: GO(4); break;                                                                \
    case 8: GO(8); break;                                                                \
    default: DH_FAIL(DH_ERR_SHAPE, name ": hidden %d too large (max 16384)", H);         \
  }

template <typename T, bool SUM>
static int rmsnorm_fwd_t(int rows, int H, const void* x, const RowSrc<T, SUM>& res, const void* gamma, float eps, void* x_out,
                         void* h, float* rstd, hipStream_t s) {
#define GO(N) rmsnorm_fwd_kernel<T, N, SUM><<<rows, ROW_THREADS, 0, s>>>((const T*)x, res, (const T*)gamma, eps, (T*)x_out, (T*)h, rstd, H)
  NCH_SWITCH("rmsnorm", H)
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_rmsnorm_fwd(int dtype, int T, int H, const void* x, const void* residual, const void* gamma,
                              float eps, void* x_out, void* h, float* rstd, void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "rmsnorm_fwd: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!x || !gamma || !h || !rstd || (residual && !x_out)) DH_FAIL(DH_ERR_INVALID_ARG, "rmsnorm_fwd: null pointer");
  hipStream_t s = (hipStream_t)stream;
  return dtype == DH_BF16 ? rmsnorm_fwd_t(T, H, x, RowSrc<bf16_t, false>{(const bf16_t*)residual}, gamma, eps, x_out, h, rstd, s)
                          : rmsnorm_fwd_t(T, H, x, RowSrc<float, false>{(const float*)residual}, gamma, eps, x_out, h, rstd, s);
}

template <typename T, bool SUM>
static int rmsnorm_bwd_t(int rows, int H, const RowSrc<T, SUM>& dy, const void* x, const void* gamma, const float* rstd,
                         const void* dres, void* dx, float* dgamma, float* partial, hipStream_t s) {
  const int nblk = (rows + norm_bwd_rpb(rows) - 1) / norm_bwd_rpb(rows);
#define GO2(N, G)                                                                                                         \
  rmsnorm_bwd_kernel<T, N, SUM, G><<<nblk, ROW_THREADS, 0, s>>>(dy, (const T*)x, (const T*)gamma, rstd, (const T*)dres, (T*)dx, \
                                                                partial, rows, H)
#define GO(N) GO2(N, 1)
  switch (norm_bwd_groups<T>(rows, H, false)) {
    case 4: GO2(1, 4); break;
    case 2: GO2(1, 2); break;
    default: NCH_SWITCH("rmsnorm", H)
  }
#undef GO
#undef GO2
  DH_LAUNCH_CHECK();
  colsum_finish_kernel<<<(H + 31) / 32, COLSUM_THREADS, 0, s>>>(partial, nblk, H, dgamma, H, nullptr);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" size_t dh_rmsnorm_bwd_ws_bytes(int T, int H) {
  size_t nblk = (size_t)(T + norm_bwd_rpb(T) - 1) / norm_bwd_rpb(T);
  return nblk * H * sizeof(float);
}

extern "C" int dh_rmsnorm_bwd(int dtype, int T, int H, const void* dy, const void* x, const void* gamma,
                              const float* rstd, const void* dres, void* dx, float* dgamma, void* ws, size_t ws_bytes,
                              void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "rmsnorm_bwd: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!dy || !x || !gamma || !rstd || !dx || !dgamma) DH_FAIL(DH_ERR_INVALID_ARG, "rmsnorm_bwd: null pointer");
  if (!ws || ws_bytes < dh_rmsnorm_bwd_ws_bytes(T, H))
    DH_FAIL(DH_ERR_WORKSPACE_TOO_SMALL, "rmsnorm_bwd: workspace %zu < %zu bytes", ws_bytes, dh_rmsnorm_bwd_ws_bytes(T, H));
  return dtype == DH_BF16
             ? rmsnorm_bwd_t(T, H, RowSrc<bf16_t, false>{(const bf16_t*)dy}, x, gamma, rstd, dres, dx, dgamma, (float*)ws, (hipStream_t)stream)
             : rmsnorm_bwd_t(T, H, RowSrc<float, false>{(const float*)dy}, x, gamma, rstd, dres, dx, dgamma, (float*)ws, (hipStream_t)stream);
}

// RMSNorm backward for callers that may not allocate (code under stream capture, serving loops): the per-block partial
// rows of the gain gradient live in a library-owned static device array instead of a caller workspace.  Every GPU holds
// its own copy of the array at its own address; the address is looked up once per device, with that device current.
#define DH_NORM_SCRATCH_BYTES (8u << 20)
static __device__ __align__(256) float dh_norm_scratch[DH_NORM_SCRATCH_BYTES / sizeof(float)];
static int norm_scratch_ptr(float** out) {
  static float* ptr[DH_MAX_DEVICES] = {};
  static std::mutex mu;
  int dev = 0;
  DH_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= DH_MAX_DEVICES) DH_FAIL(DH_ERR_UNSUPPORTED, "rmsnorm_bwd_noalloc: device index %d above %d", dev, DH_MAX_DEVICES - 1);
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    DH_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(dh_norm_scratch)));
    if (p == nullptr) DH_FAIL(DH_ERR_HIP, "rmsnorm_bwd_noalloc: the scratch array has no device address");
    ptr[dev] = (float*)p;
  }
  *out = ptr[dev];
  return DH_OK;
}

extern "C" size_t dh_rmsnorm_bwd_noalloc_max_bytes(void) { return DH_NORM_SCRATCH_BYTES; }

extern "C" int dh_rmsnorm_bwd_noalloc(int dtype, int T, int H, const void* dy, const void* x, const void* gamma,
                                      const float* rstd, const void* dres, void* dx, float* dgamma, void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "rmsnorm_bwd_noalloc: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (dtype != DH_F32 && dtype != DH_BF16) DH_FAIL(DH_ERR_INVALID_ARG, "rmsnorm_bwd_noalloc: dtype %d", dtype);
  if (T == 0) return DH_OK;
  if (!dy || !x || !gamma || !rstd || !dx || !dgamma) DH_FAIL(DH_ERR_INVALID_ARG, "rmsnorm_bwd_noalloc: null pointer");
  const size_t need = dh_rmsnorm_bwd_ws_bytes(T, H);
  if (need > DH_NORM_SCRATCH_BYTES)
    DH_FAIL(DH_ERR_WORKSPACE_TOO_SMALL, "rmsnorm_bwd_noalloc: T=%d H=%d needs %zu bytes of scratch, the static array holds %u", T, H,
            need, DH_NORM_SCRATCH_BYTES);
  float* scratch = nullptr;
  int rc = norm_scratch_ptr(&scratch);
  if (rc) return rc;
  // every partial row the finishing kernel reads is written by this call's first kernel: nothing to clear
  return dtype == DH_BF16 ? rmsnorm_bwd_t(T, H, RowSrc<bf16_t, false>{(const bf16_t*)dy}, x, gamma, rstd, dres, dx, dgamma, scratch, (hipStream_t)stream)
                          : rmsnorm_bwd_t(T, H, RowSrc<float, false>{(const float*)dy}, x, gamma, rstd, dres, dx, dgamma, scratch, (hipStream_t)stream);
}

extern "C" int dh_rope(int dtype, int T, int seq, int n_heads, int head_dim, int row_stride, float base, int inverse,
                       void* t, void* stream) {
  return dh_rope_at(dtype, T, seq, 0, n_heads, head_dim, row_stride, base, inverse, t, stream);
}

extern "C" int dh_rope_at(int dtype, int T, int seq, int pos0, int n_heads, int head_dim, int row_stride, float base, int inverse,
                          void* t, void* stream) {
  return dh_rope_pairs(dtype, DH_ROPE_HALVES, T, seq, pos0, n_heads, head_dim, row_stride, base, inverse, t, stream);
}

extern "C" int dh_rope_pairs(int dtype, int pairing, int T, int seq, int pos0, int n_heads, int head_dim, int row_stride, float base,
                             int inverse, void* t, void* stream) {
  if (pairing != DH_ROPE_HALVES && pairing != DH_ROPE_ADJACENT) DH_FAIL(DH_ERR_INVALID_ARG, "rope: unknown pairing %d", pairing);
  if (T < 0 || seq <= 0 || pos0 < 0 || n_heads <= 0 || head_dim <= 0 || head_dim % 16 || row_stride % 8 || row_stride < n_heads * head_dim)
    DH_FAIL(DH_ERR_SHAPE, "rope: T=%d seq=%d heads=%d d=%d stride=%d (d must be a multiple of 16)", T, seq, n_heads,
            head_dim, row_stride);
  if (T == 0) return DH_OK;
  if (!t) DH_FAIL(DH_ERR_INVALID_ARG, "rope: null pointer");
  const double l2b = log2((double)base), ratio = exp2(-2.0 / (double)head_dim * l2b);
  const bool four = (size_t)T * n_heads * (head_dim / 16) >= (size_t)1 << 17 && !(dtype == DH_F32 && pairing == DH_ROPE_ADJACENT);
  const size_t per_row = (size_t)(four ? (n_heads + 3) / 4 : n_heads) * (head_dim / 16), most = std::max<size_t>(1, ((size_t)1 << 31) / per_row);
  for (size_t row0 = 0; row0 < (size_t)T; row0 += most) {  // (a launch's threads are counted in 32 bits)
    const unsigned threads = (unsigned)(std::min(most, (size_t)T - row0) * per_row);
#define GO(TT, ADJ, N)                                                                                                                       \
  rope_kernel<TT, ADJ, N><<<(threads + 255) / 256, 256, 0, (hipStream_t)stream>>>((TT*)t, row0, threads, seq, pos0, n_heads, head_dim, row_stride, \
                                                                                 l2b, ratio, inverse)
#define GO2(TT, ADJ) do { if (four) GO(TT, ADJ, 4); else GO(TT, ADJ, 1); } while (0)
    if (dtype == DH_BF16) { if (pairing == DH_ROPE_ADJACENT) GO2(bf16_t, true); else GO2(bf16_t, false); }
    else { if (pairing == DH_ROPE_ADJACENT) GO(float, true, 1); else GO2(float, false); }
#undef GO2
#undef GO
    DH_LAUNCH_CHECK();
  }
  return DH_OK;
}

extern "C" int dh_swiglu_fwd(int dtype, int T, int F, const void* gu, void* a, void* stream) {
  if (T < 0 || F <= 0 || F % 8) DH_FAIL(DH_ERR_SHAPE, "swiglu_fwd: T=%d F=%d (F must be a positive multiple of 8)", T, F);
  if (T == 0) return DH_OK;
  if (!gu || !a) DH_FAIL(DH_ERR_INVALID_ARG, "swiglu_fwd: null pointer");
  size_t total = (size_t)T * (F / 8);
  dim3 g((unsigned)((total + 255) / 256)), b(256);
  if (dtype == DH_BF16)
    swiglu_fwd_kernel<bf16_t><<<g, b, 0, (hipStream_t)stream>>>((const bf16_t*)gu, (bf16_t*)a, T, F);
  else
    swiglu_fwd_kernel<float><<<g, b, 0, (hipStream_t)stream>>>((const float*)gu, (float*)a, T, F);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_swiglu_bwd(int dtype, int T, int F, const void* gu, const void* da, void* dgu, void* stream) {
  if (T < 0 || F <= 0 || F % 8) DH_FAIL(DH_ERR_SHAPE, "swiglu_bwd: T=%d F=%d (F must be a positive multiple of 8)", T, F);
  if (T == 0) return DH_OK;
  if (!gu || !da || !dgu) DH_FAIL(DH_ERR_INVALID_ARG, "swiglu_bwd: null pointer");
  size_t total = (size_t)T * (F / 8);
  dim3 g((unsigned)((total + 255) / 256)), b(256);
  if (dtype == DH_BF16)
    swiglu_bwd_kernel<bf16_t><<<g, b, 0, (hipStream_t)stream>>>((const bf16_t*)gu, (const bf16_t*)da, (bf16_t*)dgu, T, F);
  else
    swiglu_bwd_kernel<float><<<g, b, 0, (hipStream_t)stream>>>((const float*)gu, (const float*)da, (float*)dgu, T, F);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_add(int dtype, size_t n, const void* a, const void* b, void* out, void* stream) {
  if (n % 8) DH_FAIL(DH_ERR_SHAPE, "add: element count %zu must be a multiple of 8", n);
  if (!a || !b || !out) DH_FAIL(DH_ERR_INVALID_ARG, "add: null pointer");
  if (n == 0) return DH_OK;
  size_t n8 = n / 8;
  dim3 g((unsigned)((n8 + 255) / 256)), bl(256);
  if (dtype == DH_BF16)
    add_kernel<bf16_t, false><<<g, bl, 0, (hipStream_t)stream>>>((const bf16_t*)a, {(const bf16_t*)b}, (bf16_t*)out, n8);
  else
    add_kernel<float, false><<<g, bl, 0, (hipStream_t)stream>>>((const float*)a, {(const float*)b}, (float*)out, n8);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

// ------------------------------------------------------------------------------------ LayerNorm fwd
// As the RMSNorm kernel, with mean removal and a shift: optional fused x_out = x + res (+ bias), then
// mu = mean(x_out), rstd = (mean((x_out-mu)^2) + eps)^(-1/2) (two passes over the registers, so the
// variance is formed from centred values), h = gamma*(x_out-mu)*rstd + beta.
template <typename T, int NCH, bool SUM>
__global__ __launch_bounds__(ROW_THREADS) void layernorm_fwd_kernel(const T* __restrict__ x, const RowSrc<T, SUM> res,
                                                                    const T* __restrict__ res_bias, const T* __restrict__ gamma,
                                                                    const T* __restrict__ beta, float eps, T* __restrict__ x_out,
                                                                    T* __restrict__ h, float* __restrict__ mu_out,
                                                                    float* __restrict__ rstd, int H) {
  __shared__ float red[8];
  const size_t row = blockIdx.x;
  Vec8<T> v[NCH];
  float sum = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (threadIdx.x + ROW_THREADS * c) * 8;
    if (col < H) {
      v[c].load(x + row * H + col);
      if (res.present()) {
        Vec8<T> r;
        res.load(r, row * H + col);
        if (res_bias != nullptr) {
          Vec8<T> bb;
          bb.load(res_bias + col);
#pragma unroll
          for (int i = 0; i < 8; i++) r.v[i] += bb.v[i];
        }
#pragma unroll
        for (int i = 0; i < 8; i++) v[c].v[i] = to_f32(from_f32<T>(v[c].v[i] + r.v[i]));
        v[c].store(x_out + row * H + col);
      }
#pragma unroll
      for (int i = 0; i < 8; i++) sum += v[c].v[i];
    }
  }
  const float mu = block256_sum(sum, red) / (float)H;
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (threadIdx.x + ROW_THREADS * c) * 8;
    if (col < H) {
#pragma unroll
      for (int i = 0; i < 8; i++) {
        v[c].v[i] -= mu;
        ss += v[c].v[i] * v[c].v[i];
      }
    }
  }
  ss = block256_sum(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)H + eps);
  if (threadIdx.x == 0) { mu_out[row] = mu; rstd[row] = r; }
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (threadIdx.x + ROW_THREADS * c) * 8;
    if (col < H) {
      Vec8<T> g, b;
      g.load(gamma + col);
      b.load(beta + col);
#pragma unroll
      for (int i = 0; i < 8; i++) g.v[i] = g.v[i] * v[c].v[i] * r + b.v[i];
      g.store(h + row * H + col);
    }
  }
}

// ------------------------------------------------------------------------------------ LayerNorm bwd
// dx = rstd*(gh - mean(gh) - xh*mean(gh*xh)) (+ dres), gh = gamma*dy, xh = (x-mu)*rstd.  Per block one
// partial row [dgamma | dbeta] of 2H floats, reduced in fixed order by the column-sum kernels.
template <typename T, int NCH, bool SUM, int G>
__global__ __launch_bounds__(ROW_THREADS) void layernorm_bwd_kernel(const RowSrc<T, SUM> dy, const T* __restrict__ x,
                                                                    const T* __restrict__ gamma, const float* __restrict__ mu,
                                                                    const float* __restrict__ rstd, const T* __restrict__ dres,
                                                                    T* __restrict__ dx, float* __restrict__ partial, int rows, int H) {
  static_assert(G == 1 || NCH == 1, "groups are for rows of few threads");
  __shared__ float red[8];
  const int t = threadIdx.x % (ROW_THREADS / G), grp = threadIdx.x / (ROW_THREADS / G);
  Vec8<T> g[NCH];
  float dg[NCH][8], db[NCH][8];
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    int col = (t + ROW_THREADS * c) * 8;
    if (col < H) g[c].load(gamma + col);
#pragma unroll
    for (int i = 0; i < 8; i++) dg[c][i] = db[c][i] = 0.f;
  }
  const int rpb = norm_bwd_rpb(rows);
  const size_t row0 = (size_t)blockIdx.x * rpb;
  const int nrows = min(rpb, rows - (int)row0);
  Raw8<T> ndy[SUM ? 1 : NCH], nx[NCH], nres[NCH];  // the next row, as fetched (partials are fetched when their row comes up)
  auto fetch = [&](size_t row) {
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      int col = (t + ROW_THREADS * c) * 8;
      if (col < H) {
        if constexpr (!SUM) ndy[c].load(dy.p + row * H + col);
        nx[c].load(x + row * H + col);
        if (dres != nullptr) nres[c].load(dres + row * H + col);
      }
    }
  };
  fetch(row0 + min(grp, nrows - 1));
  for (int rr = 0; rr < nrows; rr += G) {
    const bool mine = G == 1 || rr + grp < nrows;  // groups without a row in the last turn make the one before again
    const size_t row = row0 + (G == 1 ? rr : min(rr + grp, nrows - 1));
    const float r = rstd[row], m = mu[row];
    Vec8<T> gh[NCH], xh[NCH];
    Raw8<T> rs[NCH];
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      const int col = (t + ROW_THREADS * c) * 8;
      if constexpr (!SUM) gh[c].from(ndy[c]);
      else if (col < H) dy.load(gh[c], row * H + col);
      xh[c].from(nx[c]);
      rs[c] = nres[c];
    }
    if (rr + G < nrows) fetch(row0 + (G == 1 ? rr + 1 : min(rr + G + grp, nrows - 1)));
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      int col = (t + ROW_THREADS * c) * 8;
      if (col < H) {
#pragma unroll
        for (int i = 0; i < 8; i++) {
          xh[c].v[i] = (xh[c].v[i] - m) * r;
          if (mine) dg[c][i] += gh[c].v[i] * xh[c].v[i];
          if (mine) db[c][i] += gh[c].v[i];
          gh[c].v[i] *= g[c].v[i];
          s1 += gh[c].v[i];
          s2 += gh[c].v[i] * xh[c].v[i];
        }
      }
    }
    s1 = rows_sum<G>(s1, red) / (float)H;
    s2 = rows_sum<G>(s2, red) / (float)H;
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      int col = (t + ROW_THREADS * c) * 8;
      if (col < H && mine) {
        Vec8<T> o;
#pragma unroll
        for (int i = 0; i < 8; i++) o.v[i] = r * (gh[c].v[i] - s1 - xh[c].v[i] * s2);
        if (dres != nullptr) {
#pragma unroll
          for (int i = 0; i < 8; i++) o.v[i] += rs[c].get(i);
        }
        o.store(dx + row * H + col);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NCH; c++) {
    store_column_sums<G>(dg[c], partial + (size_t)blockIdx.x * 2 * H, (t + ROW_THREADS * c) * 8, H);
    store_column_sums<G>(db[c], partial + (size_t)blockIdx.x * 2 * H + H, (t + ROW_THREADS * c) * 8, H);
  }
}

// ------------------------------------------------------------------------------------ GeLU (tanh form, erf form)
// 0.5 (1 + tanh u) = sigmoid(2u), so the tanh form is x * sigmoid(2u), u = sqrt(2/pi) (x + 0.044715 x^3): one
// exponential per element; its derivative is s + x s (1 - s) 2 u', s = sigmoid(2u).
__device__ __forceinline__ float gelu_tanh_inner(float x) { return 0.7978845608028654f * (x + 0.044715f * x * x * x); }
__device__ __forceinline__ float gelu_sigmoid2u(float x) { return 1.0f / (1.0f + expf(-2.0f * gelu_tanh_inner(x))); }

template <typename T, bool ERF>
__global__ void gelu_fwd_kernel(const T* __restrict__ f, T* __restrict__ a, size_t n8) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n8) return;
  Vec8<T> x;
  x.load(f + idx * 8);
#pragma unroll
  for (int i = 0; i < 8; i++)
    x.v[i] = ERF ? 0.5f * x.v[i] * (1.0f + erff(x.v[i] * 0.7071067811865476f))
                 : x.v[i] * gelu_sigmoid2u(x.v[i]);
  x.store(a + idx * 8);
}

template <typename T, bool ERF>
__global__ void gelu_bwd_kernel(const T* __restrict__ f, const T* __restrict__ da, T* __restrict__ df, size_t n8) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n8) return;
  Vec8<T> x, d;
  x.load(f + idx * 8);
  d.load(da + idx * 8);
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const float v = x.v[i];
    if (ERF) {  // Phi(v) + v phi(v)
      d.v[i] *= 0.5f * (1.0f + erff(v * 0.7071067811865476f)) + v * 0.3989422804014327f * expf(-0.5f * v * v);
    } else {
      const float sg = gelu_sigmoid2u(v);
      d.v[i] *= sg + v * sg * (1.0f - sg) * 2.0f * 0.7978845608028654f * (1.0f + 3.0f * 0.044715f * v * v);
    }
  }
  d.store(df + idx * 8);
}

// ------------------------------------------------------------------------------------ bias + residual, column sums
// out[t,:] = a[t,:] + b[t,:] + bias[:]
template <typename T, bool SUM, bool AHEAD = true>
__global__ void bias_residual_add_kernel(const T* __restrict__ a, const RowSrc<T, SUM> b, const T* __restrict__ bias,
                                         T* __restrict__ out, size_t n8, int chunks) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n8) return;
  Vec8<T> x, y, z;
  x.load(a + idx * 8);
  b.template load<AHEAD>(y, idx * 8);
  z.load(bias + (idx % chunks) * 8);
#pragma unroll
  for (int i = 0; i < 8; i++) x.v[i] += y.v[i] + z.v[i];
  x.store(out + idx * 8);
}

// dst[col] += sum over the rows of x, in one launch (or as blocks of a pair of products, g_colsum): a block owns 32 columns (4 lanes of 8), its 256 row lanes each add every 256th row,
// 8 in flight, then the lanes of a wave and the waves are added, in an order fixed by the shapes alone.
// For inputs whose two launches below (partial rows, then their sum) are mostly launches: 264 rows of 2048 columns 5.0 -> 3.9 us, 1024 of 2048 5.4 -> 4.1,
// 2048 of 768 6.4 -> 4.2; 2048 of 4096 as long, 2048 of 8192 10.9 -> 12.7, 4096 of 768 6.5 -> 9.2: few blocks, each with 64 bytes of a row.
bool dh_colsum_direct(int T, int N) { return T <= 2048 && (long long)T * N <= 8 << 20; }
template <typename T>
__global__ __launch_bounds__(1024) void colsum_direct_kernel(const T* __restrict__ x, int rows, int N, float* __restrict__ dst) {
  __shared__ float part[16][32];
  const int cl = threadIdx.x & 3, col = blockIdx.x * 32 + cl * 8;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (col < N) {
    for (int r = threadIdx.x >> 2; r < rows; r += 256 * 8) {
      Raw8<T> raw[8];
#pragma unroll
      for (int u = 0; u < 8; u++)
        if (r + 256 * u < rows) raw[u].load(x + (size_t)(r + 256 * u) * N + col);
#pragma unroll
      for (int u = 0; u < 8; u++)
        if (r + 256 * u < rows) {
          Vec8<T> v;
          v.from(raw[u]);
#pragma unroll
          for (int i = 0; i < 8; i++) s[i] += v.v[i];
        }
    }
  }
#pragma unroll
  for (int d = 4; d < 64; d <<= 1)
#pragma unroll
    for (int i = 0; i < 8; i++) s[i] += __shfl_xor(s[i], d, 64);
  if ((threadIdx.x & 63) < 4)
#pragma unroll
    for (int i = 0; i < 8; i++) part[threadIdx.x >> 6][cl * 8 + i] = s[i];
  __syncthreads();
  const int c = blockIdx.x * 32 + threadIdx.x;
  if (threadIdx.x < 32 && c < N) {
    float t = part[0][threadIdx.x];
#pragma unroll
    for (int k = 1; k < 16; k++) t += part[k][threadIdx.x];
    dst[c] += t;
  }
}

// partial[by][col] = sum of rows by*rpb .. +rpb-1 of x (ascending); a thread owns 8 columns and keeps 8 rows'
// loads in flight.  Short inputs (the row shard of sequence parallelism) take fewer rows per block so that the
// launch still covers the chip.
static inline int colsum_rows_per_block(int T) { return T >= 2048 ? 32 : 8; }
template <typename T>
__global__ __launch_bounds__(256) void colsum_rows_kernel(const T* __restrict__ x, float* __restrict__ partial, int rows, int N,
                                                          int rpb) {
  const int col = (blockIdx.x * 256 + threadIdx.x) * 8;
  if (col >= N) return;
  const int r0 = blockIdx.y * rpb, r1 = min(rows, r0 + rpb);
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r = r0; r < r1; r += 8) {
    Raw8<T> raw[8];
#pragma unroll
    for (int u = 0; u < 8; u++)
      if (r + u < r1) raw[u].load(x + (size_t)(r + u) * N + col);
#pragma unroll
    for (int u = 0; u < 8; u++)
      if (r + u < r1) {
        Vec8<T> v;
        v.from(raw[u]);
#pragma unroll
        for (int i = 0; i < 8; i++) s[i] += v.v[i];
      }
  }
  float4* p = reinterpret_cast<float4*>(partial + (size_t)blockIdx.y * N + col);
  p[0] = make_float4(s[0], s[1], s[2], s[3]);
  p[1] = make_float4(s[4], s[5], s[6], s[7]);
}

// ------------------------------------------------------------------------------------ host side (GPT-style operators)
template <typename T, bool SUM>
static int layernorm_fwd_t(int rows, int H, const void* x, const RowSrc<T, SUM>& res, const void* res_bias, const void* gamma, const void* beta,
                           float eps, void* x_out, void* h, float* mu, float* rstd, hipStream_t s) {
#define GO(N)                                                                                                               \
  layernorm_fwd_kernel<T, N, SUM><<<rows, ROW_THREADS, 0, s>>>((const T*)x, res, (const T*)res_bias, (const T*)gamma, (const T*)beta, eps, \
                                                               (T*)x_out, (T*)h, mu, rstd, H)
  NCH_SWITCH("layernorm", H)
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_layernorm_fwd(int dtype, int T, int H, const void* x, const void* residual, const void* residual_bias,
                                const void* gamma, const void* beta, float eps, void* x_out, void* h, float* mu, float* rstd,
                                void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "layernorm_fwd: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!x || !gamma || !beta || !h || !mu || !rstd || (residual && !x_out) || (residual_bias && !residual))
    DH_FAIL(DH_ERR_INVALID_ARG, "layernorm_fwd: null pointer (a residual bias needs a residual)");
  hipStream_t s = (hipStream_t)stream;
  return dtype == DH_BF16 ? layernorm_fwd_t(T, H, x, RowSrc<bf16_t, false>{(const bf16_t*)residual}, residual_bias, gamma, beta, eps, x_out, h, mu, rstd, s)
                          : layernorm_fwd_t(T, H, x, RowSrc<float, false>{(const float*)residual}, residual_bias, gamma, beta, eps, x_out, h, mu, rstd, s);
}

extern "C" size_t dh_layernorm_bwd_ws_bytes(int T, int H) { return dh_rmsnorm_bwd_ws_bytes(T, 2 * H); }

template <typename T, bool SUM>
static int layernorm_bwd_t(int rows, int H, const RowSrc<T, SUM>& dy, const void* x, const void* gamma, const float* mu, const float* rstd,
                           const void* dres, void* dx, float* dgamma, float* dbeta, float* partial, hipStream_t s) {
  const int nblk = (rows + norm_bwd_rpb(rows) - 1) / norm_bwd_rpb(rows);
#define GO2(N, G)                                                                                                                 \
  layernorm_bwd_kernel<T, N, SUM, G><<<nblk, ROW_THREADS, 0, s>>>(dy, (const T*)x, (const T*)gamma, mu, rstd, (const T*)dres, (T*)dx, partial, \
                                                                  rows, H)
#define GO(N) GO2(N, 1)
  switch (norm_bwd_groups<T>(rows, H, true)) {
    case 4: GO2(1, 4); break;
    case 2: GO2(1, 2); break;
    default: NCH_SWITCH("layernorm", H)
  }
#undef GO
#undef GO2
  DH_LAUNCH_CHECK();
  colsum_finish_kernel<<<(2 * H + 31) / 32, COLSUM_THREADS, 0, s>>>(partial, nblk, 2 * H, dgamma, H, dbeta);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_layernorm_bwd(int dtype, int T, int H, const void* dy, const void* x, const void* gamma, const float* mu,
                                const float* rstd, const void* dres, void* dx, float* dgamma, float* dbeta, void* ws,
                                size_t ws_bytes, void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "layernorm_bwd: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!dy || !x || !gamma || !mu || !rstd || !dx || !dgamma || !dbeta) DH_FAIL(DH_ERR_INVALID_ARG, "layernorm_bwd: null pointer");
  if (!ws || ws_bytes < dh_layernorm_bwd_ws_bytes(T, H))
    DH_FAIL(DH_ERR_WORKSPACE_TOO_SMALL, "layernorm_bwd: workspace %zu < %zu bytes", ws_bytes, dh_layernorm_bwd_ws_bytes(T, H));
  hipStream_t s = (hipStream_t)stream;
  return dtype == DH_BF16 ? layernorm_bwd_t(T, H, RowSrc<bf16_t, false>{(const bf16_t*)dy}, x, gamma, mu, rstd, dres, dx, dgamma, dbeta, (float*)ws, s)
                          : layernorm_bwd_t(T, H, RowSrc<float, false>{(const float*)dy}, x, gamma, mu, rstd, dres, dx, dgamma, dbeta, (float*)ws, s);
}

// ------------------------------------------------------------------------------------ behind a reduction
// The operators above with the reduction in front of them taken in: the operand comes as n_parts partial buffers.  A
// row of eight partials is 10 to 12 reads and one or two writes of memory against the two kernels' 12 to 14 and two to three; at
// 4096 x 4096 in bf16 on eight ranks, separate against one: norm forward 47 + 20 -> 60 us, norm backward 48 + 28 -> 67, add
// 47 + 16 -> 56 (5.5 to 6 TB/s all of them).  Callers have checked shapes and the operators' own pointers; the partial
// buffers are checked here, as dh_comm_standin checks them.
static int check_parts(int n_parts, const void* const* parts) {
  if (n_parts < 1 || n_parts > DH_MAX_RANKS) DH_FAIL(DH_ERR_INVALID_ARG, "reduction: %d partial buffers outside 1..%d", n_parts, DH_MAX_RANKS);
  for (int r = 0; r < n_parts; r++)
    if (!parts[r] || ((uintptr_t)parts[r] & 15)) DH_FAIL(DH_ERR_INVALID_ARG, "reduction: partial %d is null or not 16-byte aligned", r);
  return DH_OK;
}
template <typename T>
static RowSrc<T, true> sum_of(int n_parts, const void* const* parts) {
  RowSrc<T, true> src;
  for (int r = 0; r < DH_MAX_RANKS; r++) src.parts.p[r] = parts[r < n_parts ? r : 0];
  src.n = n_parts;
  return src;
}
int dh_launch_sum_rmsnorm_fwd(int dtype, int T, int H, const void* x, int n_parts, const void* const* parts, const void* gamma, float eps,
                              void* x_out, void* h, float* rstd, hipStream_t s) {
  const int rc = check_parts(n_parts, parts);
  if (rc) return rc;
  return dtype == DH_BF16 ? rmsnorm_fwd_t(T, H, x, sum_of<bf16_t>(n_parts, parts), gamma, eps, x_out, h, rstd, s)
                          : rmsnorm_fwd_t(T, H, x, sum_of<float>(n_parts, parts), gamma, eps, x_out, h, rstd, s);
}
int dh_launch_sum_rmsnorm_bwd(int dtype, int T, int H, int n_parts, const void* const* parts, const void* x, const void* gamma, const float* rstd,
                              const void* dres, void* dx, float* dgamma, float* ws, hipStream_t s) {
  const int rc = check_parts(n_parts, parts);
  if (rc) return rc;
  return dtype == DH_BF16 ? rmsnorm_bwd_t(T, H, sum_of<bf16_t>(n_parts, parts), x, gamma, rstd, dres, dx, dgamma, ws, s)
                          : rmsnorm_bwd_t(T, H, sum_of<float>(n_parts, parts), x, gamma, rstd, dres, dx, dgamma, ws, s);
}
int dh_launch_sum_layernorm_fwd(int dtype, int T, int H, const void* x, int n_parts, const void* const* parts, const void* res_bias,
                                const void* gamma, const void* beta, float eps, void* x_out, void* h, float* mu, float* rstd, hipStream_t s) {
  const int rc = check_parts(n_parts, parts);
  if (rc) return rc;
  return dtype == DH_BF16 ? layernorm_fwd_t(T, H, x, sum_of<bf16_t>(n_parts, parts), res_bias, gamma, beta, eps, x_out, h, mu, rstd, s)
                          : layernorm_fwd_t(T, H, x, sum_of<float>(n_parts, parts), res_bias, gamma, beta, eps, x_out, h, mu, rstd, s);
}
int dh_launch_sum_layernorm_bwd(int dtype, int T, int H, int n_parts, const void* const* parts, const void* x, const void* gamma,
                                const float* mu, const float* rstd, const void* dres, void* dx, float* dgamma, float* dbeta, float* ws,
                                hipStream_t s) {
  const int rc = check_parts(n_parts, parts);
  if (rc) return rc;
  return dtype == DH_BF16 ? layernorm_bwd_t(T, H, sum_of<bf16_t>(n_parts, parts), x, gamma, mu, rstd, dres, dx, dgamma, dbeta, ws, s)
                          : layernorm_bwd_t(T, H, sum_of<float>(n_parts, parts), x, gamma, mu, rstd, dres, dx, dgamma, dbeta, ws, s);
}
int dh_launch_sum_add(int dtype, int T, int H, const void* a, int n_parts, const void* const* parts, const void* bias, void* out, hipStream_t s) {
  const int rc = check_parts(n_parts, parts);
  if (rc) return rc;
  const size_t n8 = (size_t)T * (H / 8);
  const unsigned g = (unsigned)((n8 + 255) / 256);
  // Up to where all blocks are resident at once (eight a unit) a thread's loads wait for each other, beyond it the waves hide them and a thread
  // that reads one buffer after the other is kinder to the memory.  Eight ranks, 4096 columns, us, ahead / one by one: 128 rows 3.4 / 5.9, 384 4.6 / 6.9,
  // 768 8.9 / 9.3, 1024 15.0 / 11.6, 2048 31.0 / 26.7, 4096 56.9 / 53.9; four ranks: 384 rows 3.6 / 4.6, 2048 17.6 / 16.1, 4096 33.3 / 32.6.
  const bool ahead = g < 8 * 256;
#define GO(TT, AHEAD)                                                                                                              \
  do {                                                                                                                             \
    const RowSrc<TT, true> b = sum_of<TT>(n_parts, parts);                                                                         \
    if (bias) bias_residual_add_kernel<TT, true, AHEAD><<<g, 256, 0, s>>>((const TT*)a, b, (const TT*)bias, (TT*)out, n8, H / 8);  \
    else add_kernel<TT, true, AHEAD><<<g, 256, 0, s>>>((const TT*)a, b, (TT*)out, n8);                                             \
  } while (0)
  if (dtype == DH_BF16) { if (ahead) GO(bf16_t, true); else GO(bf16_t, false); }
  else { if (ahead) GO(float, true); else GO(float, false); }
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_gelu_fwd(int dtype, size_t n, const void* f, void* a, void* stream) {
  return dh_gelu_fwd_form(dtype, DH_GELU_TANH, n, f, a, stream);
}
extern "C" int dh_gelu_bwd(int dtype, size_t n, const void* f, const void* da, void* df, void* stream) {
  return dh_gelu_bwd_form(dtype, DH_GELU_TANH, n, f, da, df, stream);
}

extern "C" int dh_gelu_fwd_form(int dtype, int form, size_t n, const void* f, void* a, void* stream) {
  if (form != DH_GELU_TANH && form != DH_GELU_ERF) DH_FAIL(DH_ERR_INVALID_ARG, "gelu: unknown form %d", form);
  if (n % 8) DH_FAIL(DH_ERR_SHAPE, "gelu_fwd: element count %zu must be a multiple of 8", n);
  if (n == 0) return DH_OK;
  if (!f || !a) DH_FAIL(DH_ERR_INVALID_ARG, "gelu_fwd: null pointer");
  const size_t n8 = n / 8;
  dim3 g((unsigned)((n8 + 255) / 256)), b(256);
#define GO(TT, E) gelu_fwd_kernel<TT, E><<<g, b, 0, (hipStream_t)stream>>>((const TT*)f, (TT*)a, n8)
  if (dtype == DH_BF16) { if (form == DH_GELU_ERF) GO(bf16_t, true); else GO(bf16_t, false); }
  else { if (form == DH_GELU_ERF) GO(float, true); else GO(float, false); }
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_gelu_bwd_form(int dtype, int form, size_t n, const void* f, const void* da, void* df, void* stream) {
  if (form != DH_GELU_TANH && form != DH_GELU_ERF) DH_FAIL(DH_ERR_INVALID_ARG, "gelu: unknown form %d", form);
  if (n % 8) DH_FAIL(DH_ERR_SHAPE, "gelu_bwd: element count %zu must be a multiple of 8", n);
  if (n == 0) return DH_OK;
  if (!f || !da || !df) DH_FAIL(DH_ERR_INVALID_ARG, "gelu_bwd: null pointer");
  const size_t n8 = n / 8;
  dim3 g((unsigned)((n8 + 255) / 256)), b(256);
#define GO(TT, E) gelu_bwd_kernel<TT, E><<<g, b, 0, (hipStream_t)stream>>>((const TT*)f, (const TT*)da, (TT*)df, n8)
  if (dtype == DH_BF16) { if (form == DH_GELU_ERF) GO(bf16_t, true); else GO(bf16_t, false); }
  else { if (form == DH_GELU_ERF) GO(float, true); else GO(float, false); }
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_bias_residual_add(int dtype, int T, int H, const void* a, const void* b, const void* bias, void* out,
                                    void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "bias_residual_add: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!a || !b || !bias || !out) DH_FAIL(DH_ERR_INVALID_ARG, "bias_residual_add: null pointer");
  const size_t n8 = (size_t)T * (H / 8);
  dim3 g((unsigned)((n8 + 255) / 256)), bl(256);
  if (dtype == DH_BF16)
    bias_residual_add_kernel<bf16_t, false><<<g, bl, 0, (hipStream_t)stream>>>((const bf16_t*)a, {(const bf16_t*)b}, (const bf16_t*)bias, (bf16_t*)out, n8, H / 8);
  else
    bias_residual_add_kernel<float, false><<<g, bl, 0, (hipStream_t)stream>>>((const float*)a, {(const float*)b}, (const float*)bias, (float*)out, n8, H / 8);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" size_t dh_colsum_ws_bytes(int T, int N) {
  const size_t rpb = colsum_rows_per_block(T);
  const size_t nblk = ((size_t)T + rpb - 1) / rpb;
  return nblk * N * sizeof(float);
}

extern "C" int dh_colsum(int dtype, int T, int N, const void* x, float* out, void* ws, size_t ws_bytes, void* stream) {
  if (T < 0 || N <= 0 || N % 8) DH_FAIL(DH_ERR_SHAPE, "colsum: T=%d N=%d (N must be a positive multiple of 8)", T, N);
  if (T == 0) return DH_OK;
  if (!x || !out) DH_FAIL(DH_ERR_INVALID_ARG, "colsum: null pointer");
  if (!ws || ws_bytes < dh_colsum_ws_bytes(T, N)) DH_FAIL(DH_ERR_WORKSPACE_TOO_SMALL, "colsum: workspace %zu < %zu bytes", ws_bytes, dh_colsum_ws_bytes(T, N));
  hipStream_t s = (hipStream_t)stream;
  if (dh_colsum_direct(T, N)) {
    if (dtype == DH_BF16) colsum_direct_kernel<bf16_t><<<(N + 31) / 32, 1024, 0, s>>>((const bf16_t*)x, T, N, out);
    else colsum_direct_kernel<float><<<(N + 31) / 32, 1024, 0, s>>>((const float*)x, T, N, out);
    DH_LAUNCH_CHECK();
    return DH_OK;
  }
  const int rpb = colsum_rows_per_block(T);
  const int nblk = (T + rpb - 1) / rpb;
  float* partial = (float*)ws;
  dim3 g((N / 8 + 255) / 256, nblk);
  if (dtype == DH_BF16) colsum_rows_kernel<bf16_t><<<g, 256, 0, s>>>((const bf16_t*)x, partial, T, N, rpb);
  else colsum_rows_kernel<float><<<g, 256, 0, s>>>((const float*)x, partial, T, N, rpb);
  DH_LAUNCH_CHECK();
  colsum_finish_kernel<<<(N + 31) / 32, COLSUM_THREADS, 0, s>>>(partial, nblk, N, out, N, nullptr);
  DH_LAUNCH_CHECK();
  return DH_OK;
}
