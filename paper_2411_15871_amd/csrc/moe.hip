// Mixture-of-experts operators (paper Sec. 6.1: top-2 gating; Table 2: Router, Permute, AlltoAll,
// Group-GEMM): router, stable permutation plan, row gathers (permute, all-to-all stand-in), weighted
// combine and their backward forms.  All index work is integer and deterministic: rows are grouped by
// expert with a stable counting sort (expert ascending, then token, then k), nothing uses atomics.
#include <algorithm>
#include "common.h"

// ------------------------------------------------------------------------------------ router (M1)
// One thread per token.  Top-2 by logit, ties to the lower expert id; the two kept probabilities are the
// softmax over the two kept logits: p0 = 1/(1+exp(l1-l0)), p1 = 1-p0 computed as exp(l1-l0)/(1+exp(l1-l0)).
__global__ void moe_route_kernel(int T, int E, const float* __restrict__ logits, int32_t* __restrict__ idx,
                                 float* __restrict__ prob) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  const float* l = logits + (size_t)t * E;
  int i0 = 0, i1 = -1;
  float v0 = l[0], v1 = -INFINITY;
  for (int e = 1; e < E; e++) {
    float v = l[e];
    if (v > v0) { i1 = i0; v1 = v0; i0 = e; v0 = v; }
    else if (v > v1) { i1 = e; v1 = v; }
  }
  if (i1 < 0) {  // every other logit is minus infinity or a NaN: the lowest other expert, so that the tables stay in range
    i1 = i0 == 0 ? 1 : 0;
    v1 = l[i1];
  }
  float d = expf(v1 - v0);
  idx[2 * t] = i0;
  idx[2 * t + 1] = i1;
  prob[2 * t] = 1.0f / (1.0f + d);
  prob[2 * t + 1] = d / (1.0f + d);
}

// dlogits[t,e] = p_k (dp_k - sum_j p_j dp_j) for the two kept experts, 0 elsewhere.  A thread per element (one per token, storing E
// elements apart from its neighbours': 1500 tokens of 16 experts 3.9 us, now 2.6), up to the grid of ROUTE_BWD_BLOCKS: T * E may exceed the 2^32 - 1
// threads a launch can have (2^24 tokens of 256 experts).
#define ROUTE_BWD_BLOCKS (1u << 20)
__global__ void moe_route_bwd_kernel(int T, int E, const float* __restrict__ dprob, const int32_t* __restrict__ idx,
                                     const float* __restrict__ prob, float* __restrict__ dlogits) {
  const size_t n = (size_t)T * E, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const size_t t = i / E;
    const int e = (int)(i - t * E);
    const float p0 = prob[2 * t], p1 = prob[2 * t + 1], g0 = dprob[2 * t], g1 = dprob[2 * t + 1];
    const int i0 = idx[2 * t], i1 = idx[2 * t + 1];
    const float s = p0 * g0 + p1 * g1;
    dlogits[i] = e == i1 ? p1 * (g1 - s) : e == i0 ? p0 * (g0 - s) : 0.f;
  }
}

// ------------------------------------------------------------------------------------ permutation plan (M2, M3)
// Block e ranks the assignments (a = 2t+k, ascending) that chose expert e: a wave owns a contiguous sixteenth of them, 64 at a time, counts its
// matches from the lanes' votes, and hands out ranks behind those of the waves before it.  Bound by two rounds of loads (8192 assignments: a
// thread for each 256th of them, one load after the other, took 13 us, now 4.6).
#define RANK_WAVES 16
__global__ __launch_bounds__(64 * RANK_WAVES) void moe_rank_kernel(int n_assign, const int32_t* __restrict__ idx, int32_t* __restrict__ rank,
                                                                   int32_t* __restrict__ counts) {
  __shared__ int part[RANK_WAVES];
  const int e = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int per = ((n_assign + RANK_WAVES - 1) / RANK_WAVES + 63) / 64 * 64, a0 = min(n_assign, wave * per), a1 = min(n_assign, a0 + per);
  int count = 0;
  for (int a = a0; a < a1; a += 64 * 8) {
    int v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = a + u * 64 + lane < a1 ? idx[a + u * 64 + lane] : -1;
#pragma unroll
    for (int u = 0; u < 8; u++) count += __popcll(__ballot(v[u] == e));
  }
  if (lane == 0) part[wave] = count;
  __syncthreads();
  int r = 0;
  for (int w = 0; w < wave; w++) r += part[w];
  for (int a = a0; a < a1; a += 64 * 8) {
    int v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = a + u * 64 + lane < a1 ? idx[a + u * 64 + lane] : -1;
#pragma unroll
    for (int u = 0; u < 8; u++) {
      const unsigned long long who = __ballot(v[u] == e);
      if (v[u] == e) rank[a + u * 64 + lane] = r + __popcll(who & ((1ull << lane) - 1));
      r += __popcll(who);
    }
  }
  if (wave == RANK_WAVES - 1 && lane == 0) counts[e] = r;
}

// Sum of the values of the threads before this one, over a block of 256; `part`: 4 ints.  Ends in a barrier.
__device__ __forceinline__ int block256_before(int v, int* part) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int upto = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(upto, d, 64);
    if (lane >= d) upto += t;
  }
  if (lane == 63) part[wave] = upto;
  __syncthreads();
  for (int w = 0; w < wave; w++) upto += part[w];
  __syncthreads();
  return upto - v;
}

// Prefix sums over the experts (every block for itself, thread e for expert e): offsets[e] = first send row of expert e (send order = expert
// ascending); recv_start[e] = first receive row of expert e (receive order = [local expert][source rank], logical expert
// e = source*n_local + local); group_rows[le] = rows of local expert le.  Then, with r = rank[a]: dest[a] = send row of assignment a;
// src_tok[row] = its token; send_of_recv[j] = send row copied to receive row j; recv_of_send = the inverse.  (The prefix sums as a launch of one
// thread took 2.6-4.5 us and a gap; in here they take 0.8.)
__global__ __launch_bounds__(256) void moe_tables_kernel(int n_assign, int E, int n_local, const int32_t* __restrict__ idx, const int32_t* __restrict__ rank,
                                                         const int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                         int32_t* __restrict__ recv_start, int32_t* __restrict__ group_rows,
                                                         int32_t* __restrict__ dest, int32_t* __restrict__ src_tok,
                                                         int32_t* __restrict__ send_of_recv, int32_t* __restrict__ recv_of_send) {
  __shared__ int send0[257], recv0[257], part[4];
  const int tid = threadIdx.x, a = blockIdx.x * 256 + tid, src = E / n_local;
  const int e = a < n_assign ? idx[a] : 0, r = a < n_assign ? rank[a] : 0;
  // thread p: expert p of the send order, and the p-th expert of the receive order
  const int pe = tid < E ? tid % src * n_local + tid / src : 0;
  const int c = tid < E ? counts[tid] : 0, pc = tid < E ? counts[pe] : 0;
  const int before = block256_before(c, part), pbefore = block256_before(pc, part);
  if (tid < E) { send0[tid] = before; recv0[pe] = pbefore; }
  if (tid == E - 1) send0[E] = before + c;
  __syncthreads();
  if (blockIdx.x == 0) {
    if (tid < E) { offsets[tid] = send0[tid]; recv_start[tid] = recv0[tid]; }
    if (tid == 0) offsets[E] = send0[E];
    if (tid < n_local) group_rows[tid] = (tid + 1 < n_local ? recv0[tid + 1] : send0[E]) - recv0[tid];  // local expert tid begins with source 0
  }
  if (a >= n_assign) return;
  const int row = send0[e] + r, rr = recv0[e] + r;
  dest[a] = row;
  src_tok[row] = a >> 1;
  send_of_recv[rr] = row;
  recv_of_send[row] = rr;
}

// ------------------------------------------------------------------------------------ row movement
// out[r,:] = in[map[r],:]  (token permute, all-to-all stand-in in both directions).  One wave per row chunk.
// Bound by memory (8192 rows of 8 KiB: 21 us, 6.4 TB/s), so two movements one behind the other are one where they may be:
// via != nullptr takes row map[via[r]].
template <typename T>
__global__ __launch_bounds__(256) void gather_rows_kernel(int n_rows, int H, const T* __restrict__ in, const int32_t* __restrict__ map,
                                                          const int32_t* __restrict__ via, T* __restrict__ out) {
  const int chunks = H / 8;
  const size_t total = (size_t)n_rows * chunks, stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const size_t r = i / chunks;
    const int c = (int)(i % chunks) * 8;
    Vec8<T> v;
    v.load(in + (size_t)map[via ? via[r] : r] * H + c);
    v.store(out + r * H + c);
  }
}

// y[t,:] = w0*yp[dest[t,0],:] + w1*yp[dest[t,1],:] (+ res[t,:]); weights = prob[t,:] or 1 when prob == nullptr.
// via != nullptr: yp's rows lie in another order, row d at via[d].
template <typename T>
__global__ __launch_bounds__(256) void combine_kernel(int Ttok, int H, const T* __restrict__ yp, const int32_t* __restrict__ dest, const int32_t* __restrict__ via,
                                                      const float* __restrict__ prob, const T* __restrict__ res, T* __restrict__ y) {
  const int chunks = H / 8;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)Ttok * chunks) return;
  const size_t t = i / chunks;
  const int c = (int)(i % chunks) * 8;
  const float w0 = prob ? prob[2 * t] : 1.f, w1 = prob ? prob[2 * t + 1] : 1.f;
  Vec8<T> a, b;
  int r0 = dest[2 * t], r1 = dest[2 * t + 1];
  if (via != nullptr) { r0 = via[r0]; r1 = via[r1]; }
  a.load(yp + (size_t)r0 * H + c);
  b.load(yp + (size_t)r1 * H + c);
#pragma unroll
  for (int k = 0; k < 8; k++) a.v[k] = w0 * a.v[k] + w1 * b.v[k];
  if (res != nullptr) {
    b.load(res + t * H + c);
#pragma unroll
    for (int k = 0; k < 8; k++) a.v[k] += b.v[k];
  }
  a.store(y + t * H + c);
}

// Backward of the weighted combine: dyp[dest[t,k],:] = prob[t,k]*dy[t,:]; dprob[t,k] = <dy[t,:], yp[dest[t,k],:]>.
// One 256-thread block per token.
template <typename T>
__global__ __launch_bounds__(256) void combine_bwd_kernel(int H, const T* __restrict__ dy, const T* __restrict__ yp,
                                                          const int32_t* __restrict__ dest, const float* __restrict__ prob,
                                                          T* __restrict__ dyp, float* __restrict__ dprob) {
  __shared__ float red[8];
  const size_t t = blockIdx.x;
  const int r0 = dest[2 * t], r1 = dest[2 * t + 1];
  const float p0 = prob[2 * t], p1 = prob[2 * t + 1];
  float d0 = 0.f, d1 = 0.f;
  for (int c = threadIdx.x * 8; c < H; c += 256 * 8) {
    Vec8<T> g, a, b, o0, o1;
    g.load(dy + t * H + c);
    a.load(yp + (size_t)r0 * H + c);
    b.load(yp + (size_t)r1 * H + c);
#pragma unroll
    for (int k = 0; k < 8; k++) {
      d0 += g.v[k] * a.v[k];
      d1 += g.v[k] * b.v[k];
      o0.v[k] = p0 * g.v[k];
      o1.v[k] = p1 * g.v[k];
    }
    o0.store(dyp + (size_t)r0 * H + c);
    o1.store(dyp + (size_t)r1 * H + c);
  }
  d0 = block256_sum(d0, red);
  d1 = block256_sum(d1, red);
  if (threadIdx.x == 0) { dprob[2 * t] = d0; dprob[2 * t + 1] = d1; }
}

// ------------------------------------------------------------------------------------ host side
extern "C" int dh_moe_route(int T, int E, const float* logits, int32_t* idx, float* prob, void* stream) {
  if (T < 0 || E < 2 || E > 256) DH_FAIL(DH_ERR_SHAPE, "moe_route: T=%d E=%d (E must be 2..256)", T, E);
  if (T == 0) return DH_OK;
  if (!logits || !idx || !prob) DH_FAIL(DH_ERR_INVALID_ARG, "moe_route: null pointer");
  moe_route_kernel<<<(T + 255) / 256, 256, 0, (hipStream_t)stream>>>(T, E, logits, idx, prob);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_moe_route_bwd(int T, int E, const float* dprob, const int32_t* idx, const float* prob, float* dlogits,
                                void* stream) {
  if (T < 0 || E < 2 || E > 256) DH_FAIL(DH_ERR_SHAPE, "moe_route_bwd: T=%d E=%d (E must be 2..256)", T, E);
  if (T == 0) return DH_OK;
  if (!dprob || !idx || !prob || !dlogits) DH_FAIL(DH_ERR_INVALID_ARG, "moe_route_bwd: null pointer");
  moe_route_bwd_kernel<<<(unsigned)std::min<size_t>(((size_t)T * E + 255) / 256, ROUTE_BWD_BLOCKS), 256, 0, (hipStream_t)stream>>>(T, E, dprob, idx, prob, dlogits);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_moe_plan(int T, int E, int n_local, const int32_t* idx, const dh_moe_tables* tb, void* stream) {
  if (T < 0 || E < 2 || E > 256 || n_local < 1 || E % n_local) DH_FAIL(DH_ERR_SHAPE, "moe_plan: T=%d E=%d n_local=%d", T, E, n_local);
  if (!tb || !tb->rank || !tb->dest || !tb->src_tok || !tb->send_of_recv || !tb->recv_of_send || !tb->counts || !tb->offsets ||
      !tb->recv_start || !tb->group_rows || (T > 0 && !idx))
    DH_FAIL(DH_ERR_INVALID_ARG, "moe_plan: null pointer");
  const int n = 2 * T;
  hipStream_t s = (hipStream_t)stream;
  moe_rank_kernel<<<E, 64 * RANK_WAVES, 0, s>>>(n, idx, tb->rank, tb->counts);
  DH_LAUNCH_CHECK();
  moe_tables_kernel<<<std::max(1, (n + 255) / 256), 256, 0, s>>>(n, E, n_local, idx, tb->rank, tb->counts, tb->offsets, tb->recv_start, tb->group_rows,
                                                                 tb->dest, tb->src_tok, tb->send_of_recv, tb->recv_of_send);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_moe_gather_rows(int dtype, int n_rows, int H, const void* in, const int32_t* map, void* out, int n_blocks,
                                  void* stream) {
  return dh_launch_moe_gather_rows(dtype, n_rows, H, in, map, nullptr, out, n_blocks, (hipStream_t)stream);
}
int dh_launch_moe_gather_rows(int dtype, int n_rows, int H, const void* in, const int32_t* map, const int32_t* via, void* out, int n_blocks,
                              hipStream_t stream) {
  if (n_rows < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "moe_gather_rows: rows=%d H=%d (H must be a positive multiple of 8)", n_rows, H);
  if (n_blocks < 0 || n_blocks > 65536) DH_FAIL(DH_ERR_INVALID_ARG, "moe_gather_rows: n_blocks %d outside 0..65536", n_blocks);
  if (n_rows == 0) return DH_OK;
  if (!in || !map || !out) DH_FAIL(DH_ERR_INVALID_ARG, "moe_gather_rows: null pointer");
  size_t want = ((size_t)n_rows * (H / 8) + 255) / 256, cap = n_blocks > 0 ? (size_t)n_blocks : 4096;
  unsigned grid = (unsigned)(want < cap ? want : cap);
  if (dtype == DH_BF16) gather_rows_kernel<bf16_t><<<grid, 256, 0, stream>>>(n_rows, H, (const bf16_t*)in, map, via, (bf16_t*)out);
  else gather_rows_kernel<float><<<grid, 256, 0, stream>>>(n_rows, H, (const float*)in, map, via, (float*)out);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_moe_combine(int dtype, int T, int H, const void* yp, const int32_t* dest, const float* prob,
                              const void* residual, void* y, void* stream) {
  return dh_launch_moe_combine(dtype, T, H, yp, dest, nullptr, prob, residual, y, (hipStream_t)stream);
}
int dh_launch_moe_combine(int dtype, int T, int H, const void* yp, const int32_t* dest, const int32_t* via, const float* prob,
                          const void* residual, void* y, hipStream_t stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "moe_combine: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!yp || !dest || !y) DH_FAIL(DH_ERR_INVALID_ARG, "moe_combine: null pointer");
  unsigned grid = (unsigned)(((size_t)T * (H / 8) + 255) / 256);
  if (dtype == DH_BF16) combine_kernel<bf16_t><<<grid, 256, 0, stream>>>(T, H, (const bf16_t*)yp, dest, via, prob, (const bf16_t*)residual, (bf16_t*)y);
  else combine_kernel<float><<<grid, 256, 0, stream>>>(T, H, (const float*)yp, dest, via, prob, (const float*)residual, (float*)y);
  DH_LAUNCH_CHECK();
  return DH_OK;
}

extern "C" int dh_moe_combine_bwd(int dtype, int T, int H, const void* dy, const void* yp, const int32_t* dest, const float* prob,
                                  void* dyp, float* dprob, void* stream) {
  if (T < 0 || H <= 0 || H % 8) DH_FAIL(DH_ERR_SHAPE, "moe_combine_bwd: T=%d H=%d (H must be a positive multiple of 8)", T, H);
  if (T == 0) return DH_OK;
  if (!dy || !yp || !dest || !prob || !dyp || !dprob) DH_FAIL(DH_ERR_INVALID_ARG, "moe_combine_bwd: null pointer");
  if (dtype == DH_BF16)
    combine_bwd_kernel<bf16_t><<<T, 256, 0, (hipStream_t)stream>>>(H, (const bf16_t*)dy, (const bf16_t*)yp, dest, prob, (bf16_t*)dyp, dprob);
  else
    combine_bwd_kernel<float><<<T, 256, 0, (hipStream_t)stream>>>(H, (const float*)dy, (const float*)yp, dest, prob, (float*)dyp, dprob);
  DH_LAUNCH_CHECK();
  return DH_OK;
}
