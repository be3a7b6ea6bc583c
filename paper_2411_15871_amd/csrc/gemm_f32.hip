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

template <int NT, bool TA, bool TB, bool VEC>
__global__ __launch_bounds__(64 * F32_MAX_WAVES) void gemm_f32_kernel(int M, int N, int K, const float* __restrict__ A,
                                                                      const float* __restrict__ B, float* __restrict__ C, int accumulate,
                                                                      const float* __restrict__ bias, const int32_t* __restrict__ group_rows,
                                                                      int group_mode, int rows_in_x, int vec_out) {
  constexpr int TILE = 16 * NT, LD = TILE + 4;  // square tiles; row pitch of a partial tile
  extern __shared__ float part[];               // [waves][TILE][LD]
  const int tile_m = rows_in_x ? blockIdx.x : blockIdx.y, tile_n = rows_in_x ? blockIdx.y : blockIdx.x;
  if (group_rows != nullptr) {  // grouped: blockIdx.z = group, its rows follow those of the groups before it
    int row0 = 0;
    for (int i = 0; i < (int)blockIdx.z; i++) row0 += group_rows[i];
    const int rows = group_rows[blockIdx.z];
    if (group_mode == 2) {  // weight gradient: the group's rows are the K range
      A += (size_t)row0 * M; B += (size_t)row0 * N; C += (size_t)blockIdx.z * M * N; K = rows;
    } else {
      A += (size_t)row0 * K; B += (size_t)blockIdx.z * K * N; C += (size_t)row0 * N; M = rows;
    }
    if (rows == 0 || tile_m * TILE >= M) return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const int m0 = tile_m * TILE, n0 = tile_n * TILE;
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
  __syncthreads();
  for (int x = threadIdx.x; x < TILE * TILE / 4; x += blockDim.x) {
    const int row = x / (TILE / 4), c = (x % (TILE / 4)) * 4, gm = m0 + row, gn = n0 + c;
    if (gm >= M) continue;
    f32x4 s = *reinterpret_cast<const f32x4*>(part + row * LD + c);
    for (int w = 1; w < waves; w++) s += *reinterpret_cast<const f32x4*>(part + w * (TILE * LD) + row * LD + c);
    float* dst = C + (size_t)gm * N + gn;
    if (vec_out) {  // N a multiple of 4, C and bias 16-byte aligned
      if (gn >= N) continue;
      if (bias) s += *reinterpret_cast<const f32x4*>(bias + gn);
      if (accumulate) s += *reinterpret_cast<const f32x4*>(dst);
      *reinterpret_cast<f32x4*>(dst) = s;
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (gn + e < N) {
          const float v = bias ? s[e] + bias[gn + e] : s[e];
          dst[e] = accumulate ? dst[e] + v : v;
        }
    }
  }
}

template <bool TA, bool TB>
static int launch_f32(int M, int N, int K, int k_typical, const float* A, const float* B, float* C, bool accumulate, const float* bias,
                      const int32_t* group_rows, int group_mode, int n_groups, hipStream_t stream) {
  const int waves = std::min(F32_MAX_WAVES, std::max(1, (k_typical + 31) / 32));
  auto aligned = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  const bool vec = aligned(A) && aligned(B) && (TA ? M : K) % 4 == 0 && (TB ? K : N) % 4 == 0;
  const int vec_out = N % 4 == 0 && aligned(C) && aligned(bias);
  // 16x16 tiles load twice as much per product: they pay only while 32x32 tiles come to fewer blocks than compute units.
  const bool small = (long long)((M + 31) / 32) * ((N + 31) / 32) * n_groups < 256;
#define GO(NT, V)                                                                                                               \
  do {                                                                                                                          \
    constexpr int TILE = 16 * NT, PART = TILE * (TILE + 4) * (int)sizeof(float);                                                \
    static bool attr_set[DH_MAX_DEVICES] = {};                                                                                  \
    const int dev = dh_device_index();                                                                                          \
    if (!attr_set[dev]) {                                                                                                       \
      DH_HIP(hipFuncSetAttribute((const void*)gemm_f32_kernel<NT, TA, TB, V>, hipFuncAttributeMaxDynamicSharedMemorySize,       \
                                 F32_MAX_WAVES * PART));                                                                        \
      attr_set[dev] = true;                                                                                                     \
    }                                                                                                                           \
    const int tm = (M + TILE - 1) / TILE, tn = (N + TILE - 1) / TILE, rows_in_x = tm > 65535; /* y holds no more blocks */       \
    dim3 grid(rows_in_x ? tm : tn, rows_in_x ? tn : tm, n_groups);                                                              \
    gemm_f32_kernel<NT, TA, TB, V><<<grid, 64 * waves, waves * PART, stream>>>(M, N, K, A, B, C, accumulate ? 1 : 0, bias,      \
                                                                               group_rows, group_mode, rows_in_x, vec_out);     \
  } while (0)
  if (small) { if (vec) GO(1, true); else GO(1, false); }
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

// Grouped form: see dh_launch_gemm_grouped_bf16.  max_rows bounds every group's row count (grid size).
int dh_launch_gemm_grouped_f32(int mode, int n_groups, const int32_t* group_rows, int max_rows, int dim_a, int dim_b,
                               const float* A, const float* B, float* C, hipStream_t stream) {
  if (max_rows == 0) return DH_OK;
  if (mode == 0) return launch_f32<false, false>(max_rows, dim_b, dim_a, dim_a, A, B, C, false, nullptr, group_rows, 0, n_groups, stream);
  if (mode == 1) return launch_f32<false, true>(max_rows, dim_b, dim_a, dim_a, A, B, C, false, nullptr, group_rows, 1, n_groups, stream);
  return launch_f32<true, false>(dim_a, dim_b, max_rows, max_rows / n_groups, A, B, C, true, nullptr, group_rows, 2, n_groups, stream);
}
