#include "gemm_bf16.h"
extern template int launch_out<false, false, false>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
extern template int launch_out<false, false, true>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
extern template int launch_out<false, true, false>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
extern template int launch_out<false, true, true>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
extern template int launch_out<true, false, false>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
extern template int launch_out<true, false, true>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
extern template int launch_pair<1>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<2>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<3>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<4>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<5>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<6>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<7>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
extern template int launch_pair<8>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);

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
  int cfg;  // 0: 256x256, 2: 256x128, 5: 192x128, 4: 128x128, 6: 96x128 (one block a unit); 1: 128x128, 7: 96x128, 8: 64x128, 3: 64x64 (two)
  int bm, bn, ranges, range_k, splits, k_per_split;  // K ranges that are summed apart, and the K of one
  int k_chain;                          // the K ranges are summed one after the other in the block (0: not)
  int tail_tiles, tail_splits, tail_k;  // tail launch (0 tiles = none): its tiles, K splits and K per split
  double ns, cu_ns;                     // estimated time; what the launches keep the chip from others
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

// What a tile takes on its unit, in ns: a stage of 64 K, and what a tile costs beyond its stages and its store.  `one`: as its unit's
// only tile (a ring as deep as the LDS allows); `many`: with more tiles than units (two resident blocks a unit from 128x128 down;
// the time is then a unit's per tile).  Fitted to 37 shapes in three layouts (M 200-8192, N 512-8192, K 512-8192) with
// weights and float32 gradients that come from memory, as they do in a layer (a ring of few stages looks better with operands that stay
// in the caches: 2056x768x4096 with 64x128 tiles 22 us then, 29 in fact): the shape taken is 1.1 % slower than the best one on
// average, 13 % at worst (a shape's own time is met within 5-13 % rms).  alone: how much longer a block takes by itself
// than `many` says where that is for two resident ones, with operands just written (a weight gradient's) and with weights from memory.
struct TileCost { int cfg_one, cfg_many, bm, bn, one, fill_one, many, fill_many; double alone, alone_cold; };
static const TileCost kTiles[] = {{0, 0, 256, 256, 1270, 800, 1337, 3000, 0, 0}, {2, 2, 256, 128, 710, 1900, 760, 2000, 0, 0},
                                  {5, 5, 192, 128, 500, 2800, 620, 1600, 0, 0}, {4, 1, 128, 128, 464, 1000, 500, 100, 1.2, 1.7},
                                  {6, 7, 96, 128, 410, 1000, 370, 300, 1.5, 1.9}, {8, 8, 64, 128, 400, 400, 295, 300, 1.15, 1.4},
                                  {3, 3, 64, 64, 235, 1100, 225, 150, 0.9, 1.1}};
static const double kLaunch = 2000, kSecondLaunch = 4000, kLong = 100e3;  // ns: a launch's ramp; a dependent second launch, ramp and gap
struct TileTime { int cfg; double block; bool two; };  // ns a block takes of its unit; whether two share one
// blocks: of the whole launch; stages, store bytes an element, ranges: of one product's tiles.  (cus is passed in: asking the runtime for the current
// device costs some 40 ns each time, and a plan has seven shapes.)
static TileTime tile_time(const TileCost& c, int cus, long long blocks, int stages, double store_bytes, int chained_ranges) {
  const bool many = blocks > cus;
  double store = (double)c.bm * c.bn * store_bytes / 20;  // a unit's share of the memory's rate, 20 bytes a ns
  if (c.cfg_many == 1 && many) store *= 0.6;               // one block stores while the other multiplies
  return {many ? c.cfg_many : c.cfg_one, stages * (double)(many ? c.many : c.one) + (many ? c.fill_many : c.fill_one) + store + chained_ranges * 200.0,
          many && c.alone > 0};
}

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
// leave fewer units idle (the shapes between 64x64 and 256x128 that are no halves of one another are there for the second:
// 4000x1408x1024 17.4 -> 15.2 us with 96x128, 1504x2048x2048 21.5 -> 20.1, 8192x1280x8192 A transposed 229 -> 190 with
// 192x128).  Ranges go to blocks of their own and through the workspace (splitk_reduce_kernel), or are summed one after the
// other in the block (no workspace, no second launch; not with 256x256 tiles, whose registers hold one sum only), whichever is expected
// sooner.
//
// groups > 0: a grouped launch, `groups` products of this (average) size.  Its K is never cut (a group's extents are known on
// the device alone), so there are no ranges, and every tile shape is considered over the tiles of all groups.  b_kmajor: B's columns are
// contiguous and no part of a sum over rows (mode 0 of grouped launches, where it matters).
static GemmPlan choose_plan(int M, int N, int K, bool acc, size_t ws_bytes, int groups = 0, bool b_kmajor = false) {
  const int cus = num_cus();
  auto tiles = [&](int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  const int nkt = std::max(1, (K + 63) / 64);  // ranges are made in units of 64, a stage
  GemmPlan p = {};
  const long long t256 = tiles(256, 256), t2 = tiles(256, 128);
  const bool wide = t256 * 2 >= cus;
  const long long t = wide ? t256 : (t2 <= cus && t2 * 4 >= (long long)cus * 3) ? t2 : tiles(128, 128);
  int ranges = 1;
  if (groups == 0 && t * 4 <= cus * 3 && nkt >= 16) ranges = std::max(1, std::min((int)(cus / t), nkt / 8));
  const int per = (nkt + ranges - 1) / ranges;
  ranges = (nkt + per - 1) / per;
  p.ranges = ranges;
  p.range_k = per * 64;
  const int tail = (int)(t % cus);
  if (wide && t > cus && tail > 0 && tail * 2 <= cus && nkt >= 32 && groups == 0) {
    int ts = std::min(std::min(cus / tail, 8), nkt / 8);
    const size_t bytes = (size_t)(tail + 7) * 256 * 256 * sizeof(float);  // the launch index range is padded to a multiple of 8
    if (ws_bytes / bytes < (size_t)ts) ts = (int)(ws_bytes / bytes);
    if (ts >= 2) {
      const int kt = (nkt + ts - 1) / ts;
      p.cfg = 0; p.bm = p.bn = 256;
      p.splits = 1; p.k_per_split = nkt * 64;
      p.tail_tiles = tail; p.tail_k = kt * 64; p.tail_splits = (nkt + kt - 1) / kt;
      return p;
    }
  }
  const size_t mn = (size_t)M * N;
  auto consider = [&](const TileCost& c, int splits, bool chained, double at_most = 1.0) {  // at_most: of the best other's time
    const long long blocks = tiles(c.bm, c.bn) * splits * std::max(1, groups);
    const int stages = splits > 1 ? per : nkt;
    const TileTime tt = tile_time(c, cus, blocks, stages, splits > 1 ? 4 : acc ? 8 : 2, chained ? ranges : 0);
    double ns = (double)((blocks + cus - 1) / cus) * tt.block;
    // A long product that leaves units idle leaves them to the other strand: half of what those would have done counts.
    if (ns > kLong) ns = 0.5 * (ns + tt.block * blocks / cus);
    const double sum = splits > 1 ? kSecondLaunch + (double)mn * (4 * splits + (acc ? 8 : 2)) / 5000 : 0;  // the partials read at 5 TB/s
    ns += kLaunch + sum;
    if (p.ns != 0 && ns >= at_most * p.ns) return;
    p.ns = ns;
    p.cu_ns = tt.block * blocks / cus + kLaunch / 2 + sum;
    p.cfg = tt.cfg;
    p.bm = c.bm; p.bn = c.bn;
    p.splits = splits;
    p.k_per_split = splits > 1 ? per * 64 : nkt * 64;
    p.k_chain = chained ? per * 64 : 0;
  };
  for (const TileCost& c : kTiles) {
    // Grouped launches: the square shapes and 256x128.  64x64 where 128x128 tiles would be fewer than 96; beyond, only where they are expected to take less
    // than 0.79 of the time (4 x (1000 x 512 x 6000): the same time within the estimate's error, four times the traffic): weight gradients (76 shapes:
    // 0.77 of the time of 128x128 tiles, 0.94 at worst), and data gradients of more than a round of them (51 shapes, 0.92 on average, 0.54 to 1.44; within a
    // round the weights' rate counts, which the estimate does not see: 6, 0.81 to 1.13).  Not with weights as they are stored (B K-major, 128 bytes of a row a stage): eight
    // shapes 0.99 on average, 0.72 to 1.25.
    if (groups > 0 && c.bm != c.bn && c.bm != 256) continue;
    if (groups > 0 && c.bm == 64 && tiles(128, 128) * groups >= 96) {
      if (acc || (!b_kmajor && tiles(64, 64) * groups > cus)) consider(c, 1, false, 0.79);
      continue;
    }
    if (ranges == 1) consider(c, 1, false);
    else if (ws_bytes / (mn * sizeof(float)) >= (size_t)ranges) consider(c, ranges, false);
    if (ranges > 1 && c.bm * c.bn < 256 * 256) consider(c, 1, true);
  }
  return p;
}

// The tile shape of a data and a weight gradient that go out as one launch, each with the K ranges it has by itself (the same bits),
// summed in the block.  PAIR_APART where two launches are expected to be as fast (large products, which fill the chip by themselves): pd and pw
// are valid then, too.  PAIR_NONE: there is no launch that holds both, pd and pw are the plans of the products by themselves.
// beside: another stream's kernels run at the same time, and use the units that a launch leaves idle: what the launch takes of the chip then
// counts as much as when it ends.  (Two strands of 3 x 2727 tokens, 584 wide, heads of 64: 64x64 tiles for both gradients of the QKV projection
// end as soon as two launches of large tiles, and take 1.6 times their unit time: step 561 -> 581 us; of 3010 tokens, 1408 wide
// with heads of 64 572 -> 583; with this 564 and 528.)
// The estimate hands the blocks of the product whose blocks take longer to the units first, then the other's to whichever is free.
struct GemmShape { int M, N, K; };
enum PairChoice { PAIR_NONE, PAIR_APART, PAIR_TOGETHER };
static PairChoice choose_pair(const GemmShape& d, const GemmShape& w, int groups, bool beside, GemmPlan& pd, GemmPlan& pw, bool& w_first) {
  const int cus = num_cus(), ng = std::max(1, groups);
  pd = choose_plan(d.M, d.N, d.K, false, (size_t)-1, groups);
  pw = choose_plan(w.M, w.N, w.K, true, (size_t)-1, groups);
  if (pd.tail_tiles > 0 || pw.tail_tiles > 0) return PAIR_NONE;  // more than a round of the largest tiles, and K ranges of its own
  // A data gradient cut into many ranges would walk them one after the other, with weights that come from memory: 1344x512x4608
  // 35 us apart, 40 as one launch.  (A weight gradient's operands have just been written: 512x1024x4000 in seven ranges 26 -> 20.)
  if (pd.ranges > 4) return PAIR_NONE;
  const double shared = beside ? 0.5 : 0.0, apart = (1 - shared) * (pd.ns + pw.ns) + shared * (pd.cu_ns + pw.cu_ns);
  // Small tiles fetch their operands often, and blocks of two products at a time find less of them in the L2s, which hold 32 MiB together: beyond
  // that they take a quarter longer than estimated (7616 tokens, 304 x 2104, 64x64: 55 us against 48 apart; four sequential and two-strand steps
  // 2-3 % faster with this, 26 others the same; from 18 MB on instead, three of them 1-4 % slower).
  const double operands = 2.0 * ng * ((double)d.M * (d.N + d.K) + (double)d.K * d.N);
  double best = 0;
  for (const TileCost& c : kTiles) {
    if (c.bm * c.bn == 256 * 256) continue;
    auto blocks_of = [&](const GemmShape& g) { return (long long)((g.M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn) * ng; };
    const long long nd = blocks_of(d), nw = blocks_of(w);
    const TileTime td = tile_time(c, cus, nd + nw, (d.K + 63) / 64, 2, pd.ranges > 1 ? pd.ranges : 0);
    const TileTime tw = tile_time(c, cus, nd + nw, (w.K + 63) / 64, 8, pw.ranges > 1 ? pw.ranges : 0);
    const bool wf = tw.block > td.block;
    const long long n1 = wf ? nw : nd, n2 = wf ? nd : nw, q = n1 / cus, r = n1 % cus;
    const double t1 = wf ? tw.block : td.block, t2 = wf ? td.block : tw.block;
    const double a = q * t1, b = r > 0 ? a + t1 : a;  // the other units, and r of them, are free for the second product
    auto fits = [&](double end) {  // the second product's blocks that are through by then
      return (cus - r) * (long long)std::max(0.0, (end - a) / t2 + 1e-6) + r * (long long)std::max(0.0, (end - b) / t2 + 1e-6) >= n2;
    };
    const double even = (n1 * t1 + n2 * t2) / cus;
    double end = -1;
    for (double from : {a, b}) {
      double e = from + std::floor(std::max(0.0, even - from) / t2) * t2;
      while (!fits(e)) e += t2;
      if (end < 0 || e < end) end = e;
    }
    end = std::max(end, b);
    if (td.two) {  // two blocks share a unit: a long one goes on at half the unit's rate, and by itself once the others are through
      const double beside = std::min(t1, std::max(0.0, even - t1));
      end = std::max(end, 2 * beside + (t1 - beside) * (wf ? c.alone : c.alone_cold));
    }
    const double ns = (c.bm * c.bn < 128 * 128 && operands > 30e6 ? 1.25 : 1.0) * ((1 - shared) * (kLaunch + end) + shared * (even + kLaunch / 2));
    if (best != 0 && ns >= best) continue;
    best = ns;
    w_first = wf;
    auto take = [&](GemmPlan& p, const GemmShape& g) {
      p.cfg = td.cfg; p.bm = c.bm; p.bn = c.bn; p.splits = 1;
      p.k_per_split = std::max(1, (g.K + 63) / 64) * 64;
      p.k_chain = p.ranges > 1 ? p.range_k : 0;
    };
    take(pd, d);
    take(pw, w);
  }
  // (Nor where the weight gradient's float32 result is most of the work: a data gradient of few long blocks beside blocks that keep
  // the memory busy takes longer than by itself, T = 384, 3680 x 8496: 121 us apart, 158 as one launch.)
  // The second launch's gap is not in the estimate; of long products the forward strand's blocks use the units left idle.
  return best < apart * (apart > kLong * 1.5 ? 0.95 : beside ? 1.0 : 1.03) && 8.0 * w.M * w.N * ng / 5000 < 0.5 * best ? PAIR_TOGETHER : PAIR_APART;
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

static GemmArgs gemm_args(int M, int N, int K, const bf16_t* A, const bf16_t* B, void* C, int epi, const GemmPlan& p) {
  GemmArgs g = {};
  g.M = M; g.N = N; g.K = K; g.A = A; g.B = B; g.C = C; g.epi = epi;
  g.k_per_split = p.k_per_split; g.k_chain = p.k_chain;
  g.n_groups = 1; g.part1_bm = g.part1_bn = 256;
  return g;
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
  const int final_epi = out_f32_accumulate ? EPI_ACC_F32 : EPI_STORE_BF16;
  GemmArgs g = gemm_args(M, N, K, A, B, C, final_epi, p);
  g.bias = bias;
  int rc;
  if (p.tail_tiles > 0) {  // whole rounds with the final epilogue, then the last round's tiles with K split, then their sum
    int first, count;
    tail_range(M, N, p, first, count);
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
  if (p.splits > 1) { g.C = ws; g.epi = EPI_PARTIAL_F32; }
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
  GemmArgs g = gemm_args(M, N, K, A, B, C, out_f32_accumulate ? EPI_ACC_F32 : EPI_STORE_BF16, p);
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
  GemmArgs g = gemm_args(T, 2 * F, H, x, Wgu, gu, EPI_STORE_BF16, p);
  g.glu_mode = GLU_FWD; g.glu_f = F; g.glu_out = a;
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
  GemmArgs g = gemm_args(T, F, H, dy, Wd, dgu, EPI_STORE_BF16, p);
  g.glu_mode = GLU_BWD; g.glu_f = F; g.glu_in = gu;
  return launch_layout<false, true>(g, p, stream);
}

// Grouped GEMM with device-side row counts (expert routing is data): group z owns group_rows[z] consecutive
// rows, max_rows bounds any group (the grid is sized for it).  mode 0: C[rows,dim_b] = A[rows,dim_a] B_z[dim_a,dim_b];
// mode 1: C[rows,dim_b] = A[rows,dim_a] B_z[dim_b,dim_a]^T; mode 2: C_z[dim_a,dim_b] += A[rows,dim_a]^T B[rows,dim_b]
// (float32).  No split-K: every group is one launch slice of the same grid.
static GemmPlan grouped_plan(int mode, int n_groups, int max_rows, int dim_a, int dim_b) {  // for groups of about equal size
  const int avg = std::max(1, max_rows / n_groups);
  return mode == 2 ? choose_plan(dim_a, dim_b, avg, true, 0, n_groups) : choose_plan(avg, dim_b, dim_a, false, 0, n_groups, mode == 0);
}
void dh_gemm_grouped_bf16_tile(int mode, int n_groups, int max_rows, int dim_a, int dim_b, int* rows, int* cols) {
  const GemmPlan p = grouped_plan(mode, n_groups, max_rows, dim_a, dim_b);
  *rows = p.bm;
  *cols = p.bn;
}
static GemmArgs grouped_args(int mode, int n_groups, const int32_t* group_rows, int max_rows, int dim_a, int dim_b, const bf16_t* A, const bf16_t* B,
                             void* C, const GemmPlan& p) {
  GemmArgs g = mode == 2 ? gemm_args(dim_a, dim_b, max_rows, A, B, C, EPI_ACC_F32, p) : gemm_args(max_rows, dim_b, dim_a, A, B, C, EPI_STORE_BF16, p);
  g.group_rows = group_rows; g.group_mode = mode; g.n_groups = n_groups; g.cus = num_cus();
  g.k_per_split = g.K; g.k_chain = 0;  // no K split
  return g;
}
int dh_launch_gemm_grouped_bf16(int mode, int n_groups, const int32_t* group_rows, int max_rows, int dim_a, int dim_b,
                                const bf16_t* A, const bf16_t* B, void* C, hipStream_t stream) {
  if (dim_a % 8 || dim_b % 8) DH_FAIL(DH_ERR_SHAPE, "gemm_grouped (bf16): feature dimensions must be multiples of 8 (%d, %d)", dim_a, dim_b);
  if (max_rows == 0) return DH_OK;
  GemmPlan p = grouped_plan(mode, n_groups, max_rows, dim_a, dim_b);
  GemmArgs g = grouped_args(mode, n_groups, group_rows, max_rows, dim_a, dim_b, A, B, C, p);
  if (mode == 2) return launch_layout<true, false>(g, p, stream, n_groups);
  if (p.cfg != 0 || n_groups > 64)  // small tiles already, or too many groups for the in-kernel row scan: one launch
    return mode == 0 ? launch_layout<false, false>(g, p, stream, n_groups) : launch_layout<false, true>(g, p, stream, n_groups);
  g.group_part = 1;
  int rc = mode == 0 ? launch_layout<false, false>(g, p, stream, n_groups) : launch_layout<false, true>(g, p, stream, n_groups);
  if (rc != DH_OK) return rc;
  g.group_part = 2;
  g.M = std::min(max_rows, g.part1_bm - 1);  // a remainder is shorter than a large tile
  // The remainders' row counts are data; a group's is half a large tile on average.  Few of them leave most units idle with 128x128 tiles, each
  // walking all of K by itself: two groups, 12800 -> 4096 features, 172 us, with 64x64 tiles 95; 6400 -> 4096 80 -> 36.  (Twice as many blocks, four groups
  // of 4096 features, are as fast with either: 235 and 238 us for the whole product.)
  p.cfg = (long long)n_groups * ((g.N + 127) / 128) * 4 <= num_cus() ? 3 : 1;
  return mode == 0 ? launch_layout<false, false>(g, p, stream, n_groups) : launch_layout<false, true>(g, p, stream, n_groups);
}

// The two gradient products of a linear layer whose dY is [T, n], weight [k, n] and input [T, k]: dX[T, k] = dY * W^T and
// dW[k, n] += X^T * dY, as one launch with the bits of the two apart.  gu != nullptr: dX goes through SwiGLU's backward as in
// dh_launch_gemm_swiglu_bwd_bf16 (dX is then d(gate | up)[T, 2k]).  Products that no one launch holds go out apart, with ws as in dh_launch_gemm_bf16.
static int launch_pair_cfg(int cfg, const GemmArgs& d, const GemmArgs& w, bool w_first, hipStream_t stream, int n_groups, const BiasGrad* bias = nullptr,
                           bool* carried = nullptr) {
  switch (cfg) {
    case 1: return launch_pair<1>(d, w, w_first, stream, n_groups, bias, carried);
    case 2: return launch_pair<2>(d, w, w_first, stream, n_groups, bias, carried);
    case 3: return launch_pair<3>(d, w, w_first, stream, n_groups, bias, carried);
    case 4: return launch_pair<4>(d, w, w_first, stream, n_groups, bias, carried);
    case 5: return launch_pair<5>(d, w, w_first, stream, n_groups, bias, carried);
    case 6: return launch_pair<6>(d, w, w_first, stream, n_groups, bias, carried);
    case 7: return launch_pair<7>(d, w, w_first, stream, n_groups, bias, carried);
    case 8: return launch_pair<8>(d, w, w_first, stream, n_groups, bias, carried);
    default: DH_FAIL(DH_ERR_INVALID_ARG, "gemm pair: no kernel with tile shape %d", cfg);
  }
}
int dh_gemm_pair_shape(int n_groups, int T, int k, int n, bool beside) {
  if (T <= 0 || n_groups > 64 || k % 8 || n % 8) return 0;
  GemmPlan pd, pw;
  bool w_first;
  const int rows = n_groups > 0 ? std::max(1, T / n_groups) : T;
  return choose_pair({rows, k, n}, {k, n, rows}, n_groups, beside, pd, pw, w_first) == PAIR_TOGETHER ? pd.cfg : 0;
}
bool dh_gemm_pair_pays(int T, int k, int n, bool beside) { return dh_gemm_pair_shape(0, T, k, n, beside) != 0; }
int dh_launch_gemm_pair_bf16(int T, int k, int n, const bf16_t* dY, const bf16_t* W, const bf16_t* X, bf16_t* dX, float* dW, const bf16_t* gu,
                             bool beside, void* ws, size_t ws_bytes, hipStream_t stream) {
  return dh_launch_gemm_pair_bias_bf16(T, k, n, dY, W, X, dX, dW, gu, beside, ws, ws_bytes, stream, nullptr, nullptr);
}
int dh_launch_gemm_pair_bias_bf16(int T, int k, int n, const bf16_t* dY, const bf16_t* W, const bf16_t* X, bf16_t* dX, float* dW, const bf16_t* gu,
                                  bool beside, void* ws, size_t ws_bytes, hipStream_t stream, const BiasGrad* bias, bool* carried) {
  if (T <= 0 || k <= 0 || n <= 0 || k % 8 || n % 8) DH_FAIL(DH_ERR_SHAPE, "gemm pair (bf16): T=%d k=%d n=%d", T, k, n);
  GemmPlan pd, pw;
  bool w_first;
  if (choose_pair({T, k, n}, {k, n, T}, 0, beside, pd, pw, w_first) == PAIR_NONE) {  // e.g. dh_gemm_pair_pays was asked with another device current
    const int rc = gu != nullptr ? dh_launch_gemm_swiglu_bwd_bf16(T, k, n, dY, W, gu, dX, stream)
                                 : dh_launch_gemm_bf16(false, true, T, k, n, dY, W, dX, false, nullptr, ws, ws_bytes, stream);
    return rc ? rc : dh_launch_gemm_bf16(true, false, k, n, T, X, dY, dW, true, nullptr, ws, ws_bytes, stream);
  }
  GemmArgs d = gemm_args(T, k, n, dY, W, dX, EPI_STORE_BF16, pd), w = gemm_args(k, n, T, X, dY, dW, EPI_ACC_F32, pw);
  if (gu != nullptr) { d.glu_mode = GLU_BWD; d.glu_f = k; d.glu_in = gu; }
  d.cus = num_cus();
  return launch_pair_cfg(pd.cfg, d, w, w_first, stream, 1, bias, carried);
}
// The same for the experts' linears (group_rows as in dh_launch_gemm_grouped_bf16; T bounds the rows of all groups).
bool dh_gemm_grouped_pair_pays(int n_groups, int T, int k, int n, bool beside) { return dh_gemm_pair_shape(n_groups, T, k, n, beside) != 0; }
int dh_launch_gemm_grouped_pair_bf16(int n_groups, const int32_t* group_rows, int T, int k, int n, const bf16_t* dY, const bf16_t* W, const bf16_t* X,
                                     bf16_t* dX, float* dW, bool beside, hipStream_t stream) {
  if (T <= 0 || k <= 0 || n <= 0 || k % 8 || n % 8) DH_FAIL(DH_ERR_SHAPE, "grouped gemm pair (bf16): T=%d k=%d n=%d", T, k, n);
  GemmPlan pd, pw;
  bool w_first;
  const int avg = std::max(1, T / n_groups);
  if (choose_pair({avg, k, n}, {k, n, avg}, n_groups, beside, pd, pw, w_first) == PAIR_NONE) {
    const int rc = dh_launch_gemm_grouped_bf16(1, n_groups, group_rows, T, n, k, dY, W, dX, stream);
    return rc ? rc : dh_launch_gemm_grouped_bf16(2, n_groups, group_rows, T, k, n, X, dY, dW, stream);
  }
  return launch_pair_cfg(pd.cfg, grouped_args(1, n_groups, group_rows, T, n, k, dY, W, dX, pd),
                         grouped_args(2, n_groups, group_rows, T, k, n, X, dY, dW, pw), w_first, stream, n_groups);
}
