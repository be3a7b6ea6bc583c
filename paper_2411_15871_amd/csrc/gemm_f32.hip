// float32 GEMM for the fp32 configuration: C[M,N] (+)= opA(A) * opB(B), on the float32 matrix instruction
// (v_mfma_f32_16x16x4_f32: float32 operands, products and sums).
// Bound: at the sizes this configuration is used for (a few hundred rows and columns) a product is a chain of
// memory latencies, not a rate.  So the tiles are small (32x32, or 16x16 where
// those would leave compute units idle), their K range is cut over the waves of a block (each at
// least 32 of K, up to 16 waves) and operands go from memory straight into the fragments, two K steps ahead of their
// products; the waves' partial tiles meet in LDS and are added in wave order, so results do not depend on scheduling.
// 128x768x256: 38 -> 4.6 us, 128x256x1376: 123 -> 7.8 us against a 64x64 tile per 256 threads with the whole of K walked by each.
// Any M, N, K >= 0 is accepted; VEC: rows of both operands can be read 16 bytes (K-contiguous) or 8 bytes (K-major)
// at a time, otherwise every element is fetched and checked on its own.  Results (and a bias) likewise, 16 bytes or one element.
#include <algorithm>
#include "common.h"

#define F32_KS 16          // K of one step: four matrix instructions deep
#define F32_AHEAD 2
#define F32_MAX_WAVES 16
#define F32_PAIR_BLOCKS 2048  // blocks of a launch that two products share (see dh_gemm_f32_pair_pays)

// Fragments of one K step of an operand: v[t][e] = element (row, k0 + 4*(lane/16) + e) for the NT 16-row tiles t, where
// row = 16 t + lane%16 for a K-contiguous operand and NT*(lane%16) + t for a K-major one (two tiles interleave, so
// that a lane's pair is contiguous in memory).
template <int NT>
struct F32Frag {
  float v[NT][4];
};
template <int NT, bool KMAJOR, bool VEC>
__device__ __forceinline__ void f32_fetch(F32Frag<NT>& f, const float* __restrict__ p, int r0, int k0, int R, int K, int kend, int lane) {
  const int l16 = lane & 15, k = k0 + 4 * (lane >> 4);
  if (KMAJOR) {
    const int r = r0 + NT * l16;
#pragma unroll
    for (int e = 0; e < 4; e++) {
#pragma unroll
      for (int t = 0; t < NT; t++) f.v[t][e] = 0.f;
      if (k + e >= kend) continue;
      const float* row = p + (size_t)(k + e) * R + r;
      if (NT == 2 && VEC) {
        if (r < R) {
          const float2 x = *reinterpret_cast<const float2*>(row);
          f.v[0][e] = x.x;
          f.v[NT - 1][e] = x.y;
        }
      } else {
#pragma unroll
        for (int t = 0; t < NT; t++)
          if (r + t < R) f.v[t][e] = row[t];
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < NT; t++) {
      const int r = r0 + 16 * t + l16;
#pragma unroll
      for (int e = 0; e < 4; e++) f.v[t][e] = 0.f;
      if (r >= R) continue;
      if (VEC) {
        if (k < kend) {
          const float4 x = *reinterpret_cast<const float4*>(p + (size_t)r * K + k);
          f.v[t][0] = x.x; f.v[t][1] = x.y; f.v[t][2] = x.z; f.v[t][3] = x.w;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (k + e < kend) f.v[t][e] = p[(size_t)r * K + k + e];
      }
    }
  }
}

struct F32Args {
  int M, N, K;
  const float *A, *B;
  float* C;
  int accumulate;
  const float* bias;
  const int32_t* group_rows;
  int group_mode, vec_out, waves;  // waves: how many share K; the others of a block only help to add
  // SwiGLU in the epilogue, as in the bf16 kernels, with the bits of the row-wise operators.  Backward: the product is dA [M, N]; gate/up come from
  // glu_in [M, 2N] and d(gate), d(up) go to C [M, 2N].
  const float* glu_in = nullptr;
};
// The share of wave `wave` (of g.waves) in the tile at (m0, n0), to part.
template <int NT, bool TA, bool TB, bool VEC>
__device__ __forceinline__ void f32_share(const F32Args& g, const float* __restrict__ A, const float* __restrict__ B, int M, int K, int m0, int n0, int wave,
                                          float* part) {
  constexpr int TILE = 16 * NT, LD = TILE + 4;
  const int N = g.N, waves = g.waves, lane = threadIdx.x & 63;
  const int steps = (K + F32_KS - 1) / F32_KS, per = (steps + waves - 1) / waves;
  const int k_begin = wave * per * F32_KS, k_end = min(K, k_begin + per * F32_KS);
  f32x4 acc[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; i++)
#pragma unroll
    for (int j = 0; j < NT; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  F32Frag<NT> a[F32_AHEAD], b[F32_AHEAD];
  auto fetch = [&](int s, int k) {
    f32_fetch<NT, TA, VEC>(a[s], A, m0, k, M, K, k_end, lane);
    f32_fetch<NT, !TB, VEC>(b[s], B, n0, k, N, K, k_end, lane);
  };
#pragma unroll
  for (int s = 0; s < F32_AHEAD; s++) fetch(s, k_begin + s * F32_KS);
  for (int k = k_begin; k < k_end; k += F32_AHEAD * F32_KS) {
#pragma unroll
    for (int s = 0; s < F32_AHEAD; s++) {
#pragma unroll
      for (int e = 0; e < 4; e++)
#pragma unroll
        for (int i = 0; i < NT; i++)
#pragma unroll
          for (int j = 0; j < NT; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].v[i][e], b[s].v[j][e], acc[i][j], 0, 0, 0);
      fetch(s, k + (s + F32_AHEAD) * F32_KS);
    }
  }
  // acc[i][j][r]: row index 4*(lane/16) + r of A's tile i, column index lane%16 of B's tile j
  float* mine = part + wave * (TILE * LD);
#pragma unroll
  for (int i = 0; i < NT; i++)
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int ri = 4 * (lane >> 4) + r, cj = lane & 15;
        const int row = TA ? NT * ri + i : 16 * i + ri, col = !TB ? NT * cj + j : 16 * j + cj;
        mine[row * LD + col] = acc[i][j][r];
      }
}
// One tile; blockIdx.z is the group.
template <int NT, bool TA, bool TB, bool VEC>
__device__ __forceinline__ void f32_tile(const F32Args& g, int tile_m, int tile_n, float* part) {  // part: [waves][TILE][LD]
  constexpr int TILE = 16 * NT, LD = TILE + 4;  // square tiles; row pitch of a partial tile
  int M = g.M, K = g.K;
  const int N = g.N, waves = g.waves;
  const float *__restrict__ A = g.A, *__restrict__ B = g.B, *__restrict__ bias = g.bias;
  float* __restrict__ C = g.C;
  if (g.group_rows != nullptr) {  // grouped: its rows follow those of the groups before it
    int row0 = 0;
    for (int i = 0; i < (int)blockIdx.z; i++) row0 += g.group_rows[i];
    const int rows = g.group_rows[blockIdx.z];
    if (g.group_mode == 2) {  // weight gradient: the group's rows are the K range
      A += (size_t)row0 * M; B += (size_t)row0 * N; C += (size_t)blockIdx.z * M * N; K = rows;
    } else {
      A += (size_t)row0 * K; B += (size_t)blockIdx.z * K * N; C += (size_t)row0 * N; M = rows;
    }
    if (rows == 0 || tile_m * TILE >= M) return;
  }
  const int wave = threadIdx.x >> 6, m0 = tile_m * TILE, n0 = tile_n * TILE;
  if (wave < waves) f32_share<NT, TA, TB, VEC>(g, A, B, M, K, m0, n0, wave, part);
  __syncthreads();
  for (int x = threadIdx.x; x < TILE * TILE / 4; x += blockDim.x) {
    const int row = x / (TILE / 4), c = (x % (TILE / 4)) * 4, gm = m0 + row, gn = n0 + c;
    if (gm >= M) continue;
    f32x4 s = *reinterpret_cast<const f32x4*>(part + row * LD + c);
    for (int w = 1; w < waves; w++) s += *reinterpret_cast<const f32x4*>(part + w * (TILE * LD) + row * LD + c);
    if (g.glu_in != nullptr) {
      const size_t at = (size_t)gm * 2 * N + gn;
      if (g.vec_out) {  // glu_in aligned, too
        if (gn >= N) continue;
        const f32x4 gate = *reinterpret_cast<const f32x4*>(g.glu_in + at), up = *reinterpret_cast<const f32x4*>(g.glu_in + at + N);
        f32x4 dg, du;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          float x, y;
          swiglu_bwd_elem(gate[e], up[e], s[e], x, y);
          dg[e] = x;
          du[e] = y;
        }
        *reinterpret_cast<f32x4*>(C + at) = dg;
        *reinterpret_cast<f32x4*>(C + at + N) = du;
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (gn + e < N) swiglu_bwd_elem(g.glu_in[at + e], g.glu_in[at + N + e], s[e], C[at + e], C[at + N + e]);
      }
      continue;
    }
    float* dst = C + (size_t)gm * N + gn;
    if (g.vec_out) {  // N a multiple of 4, C and bias 16-byte aligned
      if (gn >= N) continue;
      if (bias) s += *reinterpret_cast<const f32x4*>(bias + gn);
      if (g.accumulate) s += *reinterpret_cast<const f32x4*>(dst);
      *reinterpret_cast<f32x4*>(dst) = s;
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (gn + e < N) {
          const float v = bias ? s[e] + bias[gn + e] : s[e];
          dst[e] = g.accumulate ? dst[e] + v : v;
        }
    }
  }
}

template <int NT, bool TA, bool TB, bool VEC>
__global__ __launch_bounds__(64 * F32_MAX_WAVES) void gemm_f32_kernel(const F32Args g, int rows_in_x) {
  extern __shared__ float part[];
  f32_tile<NT, TA, TB, VEC>(g, rows_in_x ? blockIdx.x : blockIdx.y, rows_in_x ? blockIdx.y : blockIdx.x, part);
}
// The gate/up projection with SwiGLU behind it: g.N = 2 * F columns [gate | up]; a block makes the tile of F columns at n0 and the one of the same outputs'
// up columns, side by side where its waves suffice (side), and stores both to C and the activation to out [M, F].
// A launch less on a chain of latencies (see dh_launch_gemm_f32_swiglu_fwd).
template <int NT>
__global__ __launch_bounds__(64 * F32_MAX_WAVES) void gemm_f32_glu_kernel(const F32Args g, float* __restrict__ out, int tiles_n, int side) {
  extern __shared__ float part[];  // [gate | up][waves][TILE][LD]
  constexpr int TILE = 16 * NT, LD = TILE + 4;
  const int F = g.N / 2, wave = threadIdx.x >> 6, m0 = blockIdx.x / tiles_n * TILE, n0 = blockIdx.x % tiles_n * TILE, half = g.waves * TILE * LD;
  if (side) {
    const int up = wave >= g.waves;
    f32_share<NT, false, false, true>(g, g.A, g.B, g.M, g.K, m0, n0 + up * F, wave - up * g.waves, part + up * half);
  } else {
    for (int up = 0; up < 2; up++) f32_share<NT, false, false, true>(g, g.A, g.B, g.M, g.K, m0, n0 + up * F, wave, part + up * half);
  }
  __syncthreads();
  for (int x = threadIdx.x; x < TILE * TILE / 4; x += blockDim.x) {
    const int row = x / (TILE / 4), c = (x % (TILE / 4)) * 4, gm = m0 + row, gn = n0 + c;
    if (gm >= g.M || gn >= F) continue;
    f32x4 s[2], a;
#pragma unroll
    for (int up = 0; up < 2; up++) {
      const float* p = part + up * half + row * LD + c;
      s[up] = *reinterpret_cast<const f32x4*>(p);
      for (int w = 1; w < g.waves; w++) s[up] += *reinterpret_cast<const f32x4*>(p + w * (TILE * LD));
      *reinterpret_cast<f32x4*>(g.C + (size_t)gm * g.N + up * F + gn) = s[up];
    }
#pragma unroll
    for (int e = 0; e < 4; e++) a[e] = swiglu_fwd_elem(s[0][e], s[1][e]);
    *reinterpret_cast<f32x4*>(out + (size_t)gm * F + gn) = a;
  }
}
// A linear's data gradient (first blocks_d blocks) and weight gradient in one launch: they read the same dY and are chains of latencies, one behind the
// other as launches of their own (128 tokens, 256 wide: 5 + 4.6, 8.2 + 5.4, 4.1 + 4.1 and 6 + 4.8 us; the two-strand step 129 -> 112 us).
template <int NTD, int NTW>
__global__ __launch_bounds__(64 * F32_MAX_WAVES) void gemm_f32_pair_kernel(const F32Args d, const F32Args w, int blocks_d, int tiles_nd, int tiles_nw) {
  extern __shared__ float part[];
  const int bx = blockIdx.x;
  if (bx < blocks_d) f32_tile<NTD, false, true, true>(d, bx / tiles_nd, bx % tiles_nd, part);
  else f32_tile<NTW, true, false, true>(w, (bx - blocks_d) / tiles_nw, (bx - blocks_d) % tiles_nw, part);
}

template <typename Kernel>
static int f32_allow_lds(Kernel kernel, bool* attr_set, int nt, int tiles = 1) {
  const int dev = dh_device_index();
  if (!attr_set[dev]) {
    DH_HIP(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, tiles * F32_MAX_WAVES * 16 * nt * (16 * nt + 4) * (int)sizeof(float)));
    attr_set[dev] = true;
  }
  return DH_OK;
}
static F32Args f32_args(int M, int N, int K, int k_typical, const float* A, const float* B, float* C, bool accumulate, const float* bias,
                        const int32_t* group_rows, int group_mode, const float* glu_in = nullptr) {
  auto aligned = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  const int waves = std::min(F32_MAX_WAVES, std::max(1, (k_typical + 31) / 32));
  return {M, N, K, A, B, C, accumulate ? 1 : 0, bias, group_rows, group_mode, N % 4 == 0 && aligned(C) && aligned(bias) && aligned(glu_in), waves, glu_in};
}
static bool f32_vec(bool ta, bool tb, const F32Args& g) {
  auto aligned = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  return aligned(g.A) && aligned(g.B) && (ta ? g.M : g.K) % 4 == 0 && (tb ? g.K : g.N) % 4 == 0;
}
// 16x16 tiles load twice as much per product: they pay only while 32x32 tiles come to fewer blocks than compute units.
static bool f32_small(int M, int N, int n_groups) { return (long long)((M + 31) / 32) * ((N + 31) / 32) * n_groups < 256; }

template <bool TA, bool TB>
static int launch_f32(int M, int N, int K, int k_typical, const float* A, const float* B, float* C, bool accumulate, const float* bias,
                      const int32_t* group_rows, int group_mode, int n_groups, hipStream_t stream, const float* glu_in = nullptr) {
  const F32Args g = f32_args(M, N, K, k_typical, A, B, C, accumulate, bias, group_rows, group_mode, glu_in);
  const bool vec = f32_vec(TA, TB, g);
#define GO(NT, V)                                                                                                         \
  do {                                                                                                                    \
    constexpr int TILE = 16 * NT, PART = TILE * (TILE + 4) * (int)sizeof(float);                                          \
    static bool attr_set[DH_MAX_DEVICES] = {};                                                                            \
    const int rc = f32_allow_lds(gemm_f32_kernel<NT, TA, TB, V>, attr_set, NT);                                           \
    if (rc) return rc;                                                                                                    \
    const int tm = (M + TILE - 1) / TILE, tn = (N + TILE - 1) / TILE, rows_in_x = tm > 65535; /* y holds no more blocks */ \
    dim3 grid(rows_in_x ? tm : tn, rows_in_x ? tn : tm, n_groups);                                                        \
    gemm_f32_kernel<NT, TA, TB, V><<<grid, 64 * g.waves, g.waves * PART, stream>>>(g, rows_in_x);                         \
  } while (0)
  if (f32_small(M, N, n_groups)) { if (vec) GO(1, true); else GO(1, false); }
  else { if (vec) GO(2, true); else GO(2, false); }
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}

int dh_launch_gemm_f32(bool ta, bool tb, int M, int N, int K, const float* A, const float* B, float* C,
                       bool accumulate, const float* bias, hipStream_t stream) {
  if (M == 0 || N == 0) return DH_OK;
  if (!ta && !tb) return launch_f32<false, false>(M, N, K, K, A, B, C, accumulate, bias, nullptr, 0, 1, stream);
  if (!ta && tb) return launch_f32<false, true>(M, N, K, K, A, B, C, accumulate, bias, nullptr, 0, 1, stream);
  if (ta && !tb) return launch_f32<true, false>(M, N, K, K, A, B, C, accumulate, bias, nullptr, 0, 1, stream);
  return launch_f32<true, true>(M, N, K, K, A, B, C, accumulate, bias, nullptr, 0, 1, stream);
}

static int f32_glu_tile(int T, int F) { return f32_small(T, 2 * F, 1) ? 16 : 32; }
static long long f32_glu_blocks(int T, int F) {
  const int tile = f32_glu_tile(T, F);
  return (long long)((T + tile - 1) / tile) * ((F + tile - 1) / tile);
}
// Whether the gate/up projection takes SwiGLU along in its launch.  Up to two blocks a unit the product waits for latencies and the second launch is the gain (us,
// apart and as one: 128 tokens, 256 -> 2 x 688, 9.1 with the gap between launches and 6.3; 333, 512 -> 2 x 1368, 25.7 and 23.4; 512, 1024 -> 2 x 1024, 36.5 and
// 33.3); beyond, twice the waves and memory a block are in each other's way (1024, 256 -> 2 x 688, 704 blocks, 17.8 and 20.1), and the two stay
// operators that a plan places.
bool dh_glu_f32_fwd_fits(int T, int F, int H) { return F % 4 == 0 && H % 4 == 0 && f32_glu_blocks(T, F) <= 512; }
// gu [T, 2F] = x * Wgu and a = silu(gate) * up; dgu [T, 2F] = SwiGLU's backward of dy * Wd^T.  The bits of the product and the row-wise operator.
int dh_launch_gemm_f32_swiglu_fwd(int T, int F, int H, const float* x, const float* Wgu, float* gu, float* a, hipStream_t stream) {
  if (T == 0) return DH_OK;
  const F32Args g = f32_args(T, 2 * F, H, H, x, Wgu, gu, false, nullptr, nullptr, 0, a);  // a: for its alignment
  const int tile = f32_glu_tile(T, F), tn = (F + tile - 1) / tile;
  const long long blocks = f32_glu_blocks(T, F);
  if (!f32_vec(false, false, g) || !g.vec_out || !dh_glu_f32_fwd_fits(T, F, H)) {  // operands that are not aligned
    const int rc = dh_launch_gemm_f32(false, false, T, 2 * F, H, x, Wgu, gu, false, nullptr, stream);
    return rc ? rc : dh_swiglu_fwd(DH_F32, T, F, gu, a, stream);
  }
  const int side = 2 * g.waves <= F32_MAX_WAVES;
#define GO(NT)                                                                                                                    \
  do {                                                                                                                            \
    constexpr int TILE = 16 * NT, PART = TILE * (TILE + 4) * (int)sizeof(float);                                                  \
    static bool attr_set[DH_MAX_DEVICES] = {};                                                                                    \
    const int rc = f32_allow_lds(gemm_f32_glu_kernel<NT>, attr_set, NT, 2);                                                       \
    if (rc) return rc;                                                                                                            \
    gemm_f32_glu_kernel<NT><<<(unsigned)blocks, 64 * g.waves * (1 + side), 2 * g.waves * PART, stream>>>(g, a, tn, side);                  \
  } while (0)
  if (tile == 16) GO(1); else GO(2);
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}
int dh_launch_gemm_f32_swiglu_bwd(int T, int F, int H, const float* dy, const float* Wd, const float* gu, float* dgu, hipStream_t stream) {
  if (T == 0) return DH_OK;
  return launch_f32<false, true>(T, F, H, H, dy, Wd, dgu, false, nullptr, nullptr, 0, 1, stream, gu);
}

// Grouped form: see dh_launch_gemm_grouped_bf16.  max_rows bounds every group's row count (grid size).
int dh_launch_gemm_grouped_f32(int mode, int n_groups, const int32_t* group_rows, int max_rows, int dim_a, int dim_b,
                               const float* A, const float* B, float* C, hipStream_t stream) {
  if (max_rows == 0) return DH_OK;
  if (mode == 0) return launch_f32<false, false>(max_rows, dim_b, dim_a, dim_a, A, B, C, false, nullptr, group_rows, 0, n_groups, stream);
  if (mode == 1) return launch_f32<false, true>(max_rows, dim_b, dim_a, dim_a, A, B, C, false, nullptr, group_rows, 1, n_groups, stream);
  return launch_f32<true, false>(dim_a, dim_b, max_rows, max_rows / n_groups, A, B, C, true, nullptr, group_rows, 2, n_groups, stream);
}

// dX[T, k] = dY[T, n] * W[k, n]^T and dW[k, n] += X[T, k]^T * dY, as one launch with the bits of the two apart (each keeps its tile and its
// waves' shares of K).  group_rows != nullptr: per group as in dh_launch_gemm_grouped_f32.  Up to a few rounds of blocks: 22 backward passes and steps of up to
// 2048 blocks took 0.86-1.01 of their time with launches apart; beyond, the products are a rate and waves that only help to add are in the way.
static long long f32_blocks(int M, int N, int n_groups) {
  const int tile = f32_small(M, N, n_groups) ? 16 : 32;
  return (long long)((M + tile - 1) / tile) * ((N + tile - 1) / tile) * n_groups;
}
bool dh_gemm_f32_pair_pays(int n_groups, int T, int k, int n) {
  return T > 0 && f32_blocks(T, k, n_groups) + f32_blocks(k, n, n_groups) <= F32_PAIR_BLOCKS;
}
// gu != nullptr (not grouped): dX goes through SwiGLU's backward as in dh_launch_gemm_f32_swiglu_bwd.
int dh_launch_gemm_f32_pair(int n_groups, const int32_t* group_rows, int T, int k, int n, const float* dY, const float* W, const float* X, float* dX,
                            float* dW, hipStream_t stream, const float* gu) {
  const F32Args d = f32_args(T, k, n, n, dY, W, dX, false, nullptr, group_rows, 1, gu);
  const F32Args w = f32_args(k, n, T, group_rows ? T / n_groups : T, X, dY, dW, true, nullptr, group_rows, 2);
  if (T <= 0 || !f32_vec(false, true, d) || !f32_vec(true, false, w) || !dh_gemm_f32_pair_pays(n_groups, T, k, n)) {
    const int rc = group_rows ? dh_launch_gemm_grouped_f32(1, n_groups, group_rows, T, n, k, dY, W, dX, stream)
                   : gu       ? dh_launch_gemm_f32_swiglu_bwd(T, k, n, dY, W, gu, dX, stream)
                              : dh_launch_gemm_f32(false, true, T, k, n, dY, W, dX, false, nullptr, stream);
    if (rc) return rc;
    return group_rows ? dh_launch_gemm_grouped_f32(2, n_groups, group_rows, T, k, n, X, dY, dW, stream)
                      : dh_launch_gemm_f32(true, false, k, n, T, X, dY, dW, true, nullptr, stream);
  }
  const int waves = std::max(d.waves, w.waves);
#define GO(NTD, NTW)                                                                                                          \
  do {                                                                                                                        \
    constexpr int TD = 16 * NTD, TW = 16 * NTW;                                                                               \
    static bool attr_set[DH_MAX_DEVICES] = {};                                                                                \
    const int rc = f32_allow_lds(gemm_f32_pair_kernel<NTD, NTW>, attr_set, NTD > NTW ? NTD : NTW);                            \
    if (rc) return rc;                                                                                                        \
    const int lds = std::max(d.waves * TD * (TD + 4), w.waves * TW * (TW + 4)) * (int)sizeof(float);                          \
    const int nd = (k + TD - 1) / TD, nw = (n + TW - 1) / TW, blocks_d = (T + TD - 1) / TD * nd, blocks_w = (k + TW - 1) / TW * nw; \
    gemm_f32_pair_kernel<NTD, NTW><<<dim3(blocks_d + blocks_w, 1, n_groups), 64 * waves, lds, stream>>>(d, w, blocks_d, nd, nw); \
  } while (0)
  const bool sd = f32_small(T, k, n_groups), sw = f32_small(k, n, n_groups);
  if (sd && sw) GO(1, 1);
  else if (sd) GO(1, 2);
  else if (sw) GO(2, 1);
  else GO(2, 2);
#undef GO
  DH_LAUNCH_CHECK();
  return DH_OK;
}
