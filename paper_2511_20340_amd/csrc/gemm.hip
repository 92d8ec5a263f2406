// bf16 linear layers: kernel choice, split-K finish, weight packing (the kernels: gemm_ring.h, gemm_block.h, gemm_stream.hip).
#include "gemm_common.h"

#include <algorithm>
#include <cmath>

namespace sf {
namespace {

// The second launch of a layer whose K is split: adds a row's partials in split order, applies the fused norm's row
// factor and the epilogue.  One thread per 8 output columns of a row; partials are read once, whole lines, by every
// compute unit.  The alternative, one launch in which the last workgroup of a tile to arrive adds the tile's partials
// behind write-through stores and an agent-scope ticket, costs 8 us at 5 MB of partials and 20 us at 21 MB where
// this launch costs 5 and 15: 160 x 2048 x 2048 in 4 splits 15.8 -> 13.8 us, 5 x 4096 x 14336 in 8 splits
// 32.3 -> 26.9 us, 160 x 2048 x 4096 in 8 splits 31.2 -> 20.0 us.
__global__ __launch_bounds__(256) void split_finish_kernel(const float *__restrict__ partial,
                                                           const float *__restrict__ ssq_part, const Epilogue e,
                                                           int split, int M, int N, int K, float eps) {
  const int cols8 = (e.glu ? N / 2 : N) / 8;
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= M * cols8) return;
  const int row = idx / cols8, col = (idx - row * cols8) * 8;
  const float *p = partial + (size_t)row * N + (e.glu ? (col >> 4) * 32 + (col & 15) : col);
  const size_t step = (size_t)M * N;
  float r[8], up[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = up[i] = 0.f;
#pragma unroll 4
  for (int s = 0; s < split; ++s) {
    float q[8];
    load_n(p + s * step, q, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] += q[i];
    if (e.glu) {
      load_n(p + s * step + 16, q, 1);
#pragma unroll
      for (int i = 0; i < 8; ++i) up[i] += q[i];
    }
  }
  if (ssq_part) {
    float t = 0.f;
    for (int s = 0; s < split; ++s) t += ssq_part[(size_t)s * M + row];
    const float rinv = 1.0f / sqrtf(t / (float)K + eps);
#pragma unroll
    for (int i = 0; i < 8; ++i) { r[i] *= rinv; up[i] *= rinv; }
  }
  if (e.glu) {
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = r[i] / (1.0f + __expf(-r[i])) * up[i];
    store_n(reinterpret_cast<bf16_t *>(e.y) + (size_t)row * (N >> 1) + col, r, e.vec);
    return;
  }
  finish_row8(e, row, col, N, r);
}

// row-major [N][K] -> packed units; one thread per 16-byte operand register
// glu_F > 0: W is [2F][K] = [gate; up] and packed row block nb holds gate rows 16nb..16nb+15 followed
// by up rows 16nb..16nb+15 (see the SwiGLU epilogue)
// col_gain != nullptr: column k of W is multiplied by col_gain[k] (rounded to bf16 again): the gain
// vector of the RMSNorm in front of this layer, folded in for the fused norm
__global__ void pack_weight_kernel(const bf16_t *__restrict__ W, uint4 *__restrict__ P, int N, int K, size_t units,
                                   int glu_F, const bf16_t *__restrict__ col_gain) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= units) return;
  const int lane = idx & 63;
  const size_t u = idx >> 6;
  const int k_steps = (K + 15) >> 4;
  const int kstep = u % k_steps;
  const int nb = u / k_steps;
  int row = nb * 32 + (lane & 31);
  const int k0 = kstep * 16 + (lane >> 5) * 8;
  if (glu_F > 0) {
    const int within = lane & 31, f = nb * 16 + (within & 15);
    row = f < glu_F ? (within < 16 ? f : glu_F + f) : N;
  }
  uint32_t w[4] = {0, 0, 0, 0};
  if (row < N)
    for (int e = 0; e < 8; ++e)
      if (k0 + e < K) {
        bf16_t v = W[(size_t)row * K + k0 + e];
        if (col_gain) v = f2bf(bf2f(v) * bf2f(col_gain[k0 + e]));
        w[e >> 1] |= (uint32_t)v << ((e & 1) * 16);
      }
  P[idx] = make_uint4(w[0], w[1], w[2], w[3]);
}

// Tile configurations: rows per workgroup TM*32, columns NW*32 (one 32-column block per wave).
// The ring kernel's 1-14: gemm_tiles_*.hip (11-14: tall tiles for wide layers, see pick_large; 9, the three-slot form of 10,
// is chosen by no rule).
// A sixth template argument of 1 selects the hand-pinned issue order of the slice (same arithmetic, same
// bits).  Measured against the compiler's order on 27 shapes x splits {1, 2, 4}: 2-12 % faster on the 96-row
// tiles and the 128-row tiles, up to 17 % on the 64 x 256 tile, 9-60 % on the two-slot 160 x 256 tile (which
// then beats the three-slot one in the compiler's order by 1-4 % everywhere; pinned, the three-slot one is
// 1-5 % slower than unpinned); under the pinned order two ring slots beat three by 1-5 % on the 128-row
// tiles, four slots stay best on the 96-row ones; the 160 x 128 tile fits the pinned order with two slots and
// gains 5-10 % (15-22 % with the fused norm, whose extra cost drops to the 1-9 % of the other tiles).  The
// 32- and 64-row tiles move by +-3 % either way and stay as they were, the 192-row tile is faster in the
// compiler's order, and the taller tiles have no registers left for the pinned one.  An argument of 2 pins
// only where a slice's loads and LDS stores are issued: the plain 320- and 256-row kernels (LM heads) are
// 6-8 % faster with it, also inside whole steps; the 320-row kernel with the fused norm measured 3 % faster
// alone but 3.7 % slower as the gate/up product inside whole steps, so the fused-norm kernels keep the
// compiler's order (seventh argument).
// 15-31: the block and panel kernels' (gemm_block.hip, gemm_panel.hip); forced on a layer that they do not take they stand
// for tile 10.
constexpr int N_TILES = 31, N_RING_TILES = 14, N_MODEL_TILES = 10;
constexpr int TILE_TM[N_TILES + 1] = {0, 1, 2, 3, 4, 5, 2, 3, 4, 5, 5, 10, 8, 7, 6, 10, 8, 6, 4, 4, 2, 5, 5, 2, 1, 1, 4, 5, 5, 10, 8, 6};

// the block kernel's direct loads move 16 bytes at a time; the ring kernel takes rows at any address
bool rows_aligned(const GemmArgs &a) { return (uintptr_t)a.x % 16 == 0; }

// Heuristic choice (used when nothing was measured for the shape).  What the sweeps on MI355X
// showed: a compute unit draws at most ~20-40 B/clk from L2, so both the weight re-reads of the
// M-tiles and the activation re-reads of the column tiles count; ~224 workgroups fill the chip;
// splitting K costs a partial-tile round trip and a serial tail, so it is used only when the
// unsplit grid is too small and K is long.
constexpr int WG_FULL = 224, WG_SPLIT = 160;
constexpr size_t REREAD_CAP = 384u << 20;

int pow2floor(int v) { int p = 1; while (p * 2 <= v) p *= 2; return p; }

// Large M (>= 384 rows: the batch-256 and batch-128 workloads).  There the choice is a trade between
// operand traffic per compute unit, MFMA time per compute unit, how evenly the workgroups divide over
// 256 CUs and the cost of splitting K, and a cost model ranks the candidates better than rules.  Per
// workgroup: operand bytes (BM + BN) * K/split * 2 and 2 * BM * BN * K/split flop; a CU works through
// ceil(workgroups / 256) of them at ~88 GB/s of operand intake and ~9.5 TFLOP/s, the two hardly
// overlapping (the shorter one counts for 86 %); ~8 us of launch and drain; a split costs ~8 us plus its
// partial tiles (M * N * 4 * split bytes) at ~1.1 TB/s.  The constants and the per-tile factors were
// searched for the smallest regret of the choice, with the model's own error held at 13 % rms, over
// sweeps of all tiles x splits {1,2,4} (medians of interleaved repeats) of 30 shapes on MI355X: the 8B
// layers at 384 ... 1792 rows, the 14B layers at 448 ... 896 rows and the two LM heads; the factors of the
// tiles whose issue order was pinned later (4, 5, 7, 8, 10) were lowered by what the pinning gained in a repeat of
// the same sweeps.  Over the 32 shapes of that repeat the choice (this model, then the tall-tile rule) was
// the fastest configuration of the ring kernel at every shape.  Since then the second launch of a split has become cheaper
// than the model has it, and most of these layers run on the block kernel (pick_any).  The split is still decided here, as
// it fixes the order of a layer's sums; the tiles serve the layers that the block kernel does not take.
double model_us(int M, int N, int K, int tile, int split) {
  static const double factor[N_MODEL_TILES + 1] = {0, 1.0, 1.022, 1.005, 1.015, 1.080, 1.0, 0.889, 0.842, 0.938, 0.910};
  const int BM = TILE_TM[tile] * 32, BN = tile >= 6 ? 256 : 128;
  const double tiles = (double)((M + BM - 1) / BM) * ((N + BN - 1) / BN) * split;
  const double per_cu = std::ceil(tiles / 256.0), ks = (double)K / split;
  const double t_mem = per_cu * (BM + BN) * ks * 2.0 / 87.6e9;
  const double t_mma = per_cu * 2.0 * BM * BN * ks / 9.5e12;
  const double t_hbm = (double)N * K * 2.0 / 4.7e12;
  const double t = std::max({t_mem, t_mma, t_hbm}) + 0.86 * std::min(t_mem, t_mma);
  const double t_split = split > 1 ? 8.1 + (double)M * N * 4.0 * split / 1.08e12 * 1e6 : 0.0;
  return (t * 1e6 + 8.4 + t_split) * factor[tile];
}

GemmConfig pick(int M, int N, int K, size_t ws_bytes, int fixed_split);

GemmConfig pick_large(int M, int N, int K, size_t ws_bytes, int fixed_split) {
  const int KT = (K + BK - 1) / BK;
  GemmConfig best = {0, 0};
  double best_us = 0;
  for (int split = 1; split <= 4; split *= 2) {
    if (fixed_split > 0 && split != fixed_split) continue;
    if (split > 1 && KT / split < 8) continue;
    for (int tile = 2; tile <= N_MODEL_TILES; ++tile) {
      if (tile == 6) continue;  // 64 x 256: never competitive at this many rows
      if (split > 1) {
        const Plan p = make_plan(M, N, K, TILE_TM[tile] * 32, tile >= 6 ? 256 : 128, split);
        if (!plan_fits(p, TILE_TM[tile] * 32, (const void *)1, ws_bytes)) continue;
      }
      const double us = model_us(M, N, K, tile, split);
      if (best.tile == 0 || us < best_us) { best = {tile, split}; best_us = us; }
    }
  }
  // Wide layers (gate/up, LM heads): where the model lands on an unsplit 256-column tile, a taller tile of
  // the same width (192 ... 320 rows: the weights pass through fewer M-tiles) is 4-18 % faster in every
  // sweep, provided it still gives ~200 workgroups and divides M with little padding.  Among those the
  // one with the least work per compute unit is taken: rounds of 256 workgroups x (rows per workgroup + 32
  // for what a workgroup costs besides its rows), weighted by the padded share of its rows -- the order the
  // sweeps show.
  if (best.split == 1 && best.tile >= 7 && best.tile <= N_MODEL_TILES) {
    int tall = 0;
    double tall_cost = 0;
    for (int tile = N_MODEL_TILES + 1; tile <= N_RING_TILES; ++tile) {  // 320, 256, 224, 192 rows
      const int bm = TILE_TM[tile] * 32, tiles_m = (M + bm - 1) / bm, pad = tiles_m * bm - M;
      const long wgs = (long)tiles_m * ((N + 255) / 256);
      if (wgs < 200 || pad * 100 > 8 * M) continue;
      const double cost = (double)((wgs + 255) / 256) * (bm + 32) * (M + pad) / M;
      if (tall == 0 || cost < tall_cost) { tall = tile; tall_cost = cost; }
    }
    if (tall) best.tile = tall;
  }
  return best;
}

GemmConfig pick(int M, int N, int K, size_t ws_bytes, int fixed_split) {
  if (M >= 384 && (fixed_split <= 0 || fixed_split == 1 || fixed_split == 2 || fixed_split == 4)) {
    const GemmConfig c = pick_large(M, N, K, ws_bytes, fixed_split);
    if (c.tile > 0) return c;
  }
  const int KT = (K + BK - 1) / BK;
  const size_t wbytes = (size_t)N * K * 2;
  const int max_tm = std::min(5, (M + 31) / 32);
  const int cols4 = (N + 127) / 128, cols8 = (N + 255) / 256;
  auto reread_ok = [&](int tm) {
    const int tiles_m = (M + tm * 32 - 1) / (tm * 32);
    return tm == max_tm || (size_t)tiles_m * wbytes <= REREAD_CAP;
  };
  auto with_waves = [&](int tm, int split) {  // 8-wave workgroups when the grid stays full
    const int tiles_m = (M + tm * 32 - 1) / (tm * 32);
    if (!(tm >= 2 && split == 1 && tiles_m * cols8 >= WG_FULL)) return tm;
    return tm == 5 ? 10 : tm + 4;  // of the two 160 x 256 tiles the two-slot one is 1-4 % faster at every shape measured
  };
  auto fits = [&](int tm, int split) {
    if (split == 1) return true;
    const Plan p = make_plan(M, N, K, tm * 32, 128, split);
    return plan_fits(p, tm * 32, (const void *)1, ws_bytes);
  };
  auto tiles_of = [&](int tm) { return (M + tm * 32 - 1) / (tm * 32); };
  auto trim = [&](int tm) {  // fewest padded rows among the block heights with the same tile count
    while (tm > 1 && tiles_of(tm - 1) == tiles_of(tm)) --tm;
    return tm;
  };
  if (fixed_split <= 1) {
    for (int tm = max_tm; tm >= 1; --tm)
      if (tiles_of(tm) * cols4 >= WG_FULL && reread_ok(tm)) return {with_waves(trim(tm), 1), 1};
    if (fixed_split == 1) {
      for (int tm = 1; tm <= max_tm; ++tm)
        if (reread_ok(tm)) return {tm, 1};
      return {max_tm, 1};
    }
  }
  // partial tiles cost 8 bytes per output element and split (written, then read): keep that
  // below the weight bytes, and at least 8 K slices per workgroup
  const int split_cap = std::max(1, std::min({16, pow2floor(std::max(1, K / (4 * std::max(M, 1)))), KT / 8}));
  // weights that stay in L2 are cheap to re-read: there small row blocks come first (less split
  // for the same number of workgroups); larger ones are tried from the tallest block down
  const bool small_w = wbytes <= (24u << 20);
  GemmConfig best = {1, 1};
  int best_wgs = 0;
  for (int i = 0; i < max_tm; ++i) {
    const int tm = small_w ? 1 + i : max_tm - i;
    const int wgs = tiles_of(tm) * cols4;
    int sp = 1;
    if (fixed_split > 1) {
      sp = fixed_split;
    } else {
      while (wgs * sp < WG_SPLIT && sp * 2 <= split_cap) {
        if (wgs * sp >= 128 && KT / sp <= 32) break;  // enough workgroups for a short K loop
        sp *= 2;
      }
      while (sp > 1 && !fits(tm, sp)) sp /= 2;
    }
    if (!reread_ok(tm)) continue;
    if (wgs * sp >= WG_SPLIT) return {trim(tm), sp};
    if (wgs * sp > best_wgs) { best = {tm, sp}; best_wgs = wgs * sp; }
  }
  return best;
}

// What a launch of a layer takes on MI355X, in us; the measured side of the choice below.  A compute unit works through its
// workgroups one after the other (`least`: so many count where fewer do not keep it busy), each a fixed part and a part per
// 64 positions of K (with the fused norm a little more); the weights have to come from memory, which overlaps a good half of
// the shorter of the two; a split adds the second launch and its partial rows, unless groups of waves share it.  The ring
// and block kernels' tiles x splits 1 to 8 were measured on 440 shapes (the 1B, 8B and 14B layers and heads at 40 to 2304
// rows, weights cold, medians of interleaved repeats) and the constants fitted to them: 4.8 % rms.  Since float outputs leave
// in whole lines, launches of the tall tiles are up to 12 % faster than this; constants fitted anew choose no better.  (Tile
// 20's norm by hand: its waves have one row block, and the squares of one chunk wait for each other.)  The panel kernel's
// tiles (15-17, 26-28) were fitted to 360 shapes of 40 to 2304 rows, weights rotated through 600 MB, 6 to 9 % rms; their
// norm is a launch in front, priced 4 us above what it takes by itself: so much more a launch costs in the chain of a step.
// All of these have K >= 2048.  On 420 shapes of 2 to 16 slices of K (170 to 3000 rows, 1024 to 16384 columns) the prices hold
// but for tile 26 and the tall ring tiles, which have another line there (cost_us); with it the choice is 1.1 % slower than
// the fastest tile of each, 5 % without (900 x 16384 x 128 took 20.2 us for 13.5).
// Tiles 29-31 have one too: 483 x 9136 x 64 with the norm takes 14.1 us on tile 29, 9.0 on 18 (up to 4 us more than the line
// says, as tile 18 is there, which keeps its price: beside the ring kernel's, short as well, it holds).
// Tile 18 has one row for both kernels: the constants are the block kernel's, which it runs on with the norm; without it the
// panel kernel's times are 0.82 to 1.07 of the formula's (13 shapes of 192 to 2048 rows, 7 % rms).
struct TileCost {
  int bm, bn, groups;
  float slice, fixed, least, norm;
};
constexpr TileCost TILE_COST[N_TILES + 1] = {
    {},
    {32, 128, 1, 0.241f, 1.2f, 1.19f, 0.000f}, {64, 128, 1, 0.304f, 2.0f, 1.27f, 0.018f},
    {96, 128, 1, 0.385f, 3.2f, 1.11f, 0.034f}, {128, 128, 1, 0.493f, 2.9f, 1.09f, 0.045f},
    {160, 128, 1, 0.636f, 3.0f, 1.06f, 0.044f}, {64, 256, 1, 0.540f, 2.7f, 1.10f, 0.002f},
    {96, 256, 1, 0.708f, 5.7f, 1.00f, 0.026f}, {128, 256, 1, 0.849f, 4.1f, 1.00f, 0.044f},
    {160, 256, 1, 1.105f, 4.5f, 1.00f, 0.086f}, {160, 256, 1, 1.105f, 4.5f, 1.00f, 0.086f},
    {320, 256, 1, 2.072f, 2.4f, 1.00f, 0.333f}, {256, 256, 1, 1.593f, 3.3f, 1.00f, 0.302f},
    {224, 256, 1, 1.560f, 4.4f, 1.00f, 0.095f}, {192, 256, 1, 1.167f, 6.0f, 1.00f, 0.096f},
    {320, 256, 1, 1.403f, 11.3f, 1.00f, 6.2f}, {256, 256, 1, 1.238f, 8.9f, 1.00f, 7.0f},
    {192, 256, 1, 1.071f, 7.1f, 1.00f, 7.2f}, {128, 256, 1, 0.744f, 4.5f, 1.00f, 0.081f},
    {128, 64, 1, 0.293f, 1.7f, 1.12f, 0.041f}, {64, 64, 1, 0.199f, 1.1f, 1.12f, 0.140f},
    {160, 64, 1, 0.392f, 3.2f, 1.00f, 0.081f}, {160, 128, 1, 0.548f, 4.9f, 1.00f, 0.117f},
    {64, 64, 2, 0.469f, 0.2f, 1.00f, 0.083f}, {32, 64, 4, 0.737f, 0.0f, 1.00f, 0.089f},
    {32, 64, 2, 0.348f, 0.1f, 1.00f, 0.038f}, {128, 128, 1, 0.526f, 1.1f, 1.00f, 8.5f},
    {160, 128, 1, 0.486f, 1.9f, 1.63f, 7.8f}, {160, 128, 1, 0.509f, 4.3f, 1.00f, 7.0f},
    {320, 256, 1, 1.691f, 2.6f, 1.00f, 0.230f}, {256, 256, 1, 1.317f, 3.2f, 1.00f, 0.232f}, {192, 256, 1, 1.027f, 3.7f, 1.00f, 0.143f},
};
double cost_us(int M, int N, int K, GemmConfig c, int norm) {
  const TileCost &t = TILE_COST[c.tile];
  const int KT = (K + BK - 1) / BK, kps = (KT + c.split - 1) / c.split, split = (KT + kps - 1) / kps;
  const int tiles_m = (M + t.bm - 1) / t.bm, units = (N + t.bn - 1) / t.bn * (t.groups > 1 ? 1 : split);
  const int per_cu = ((units + XCDS - 1) / XCDS * tiles_m + 31) / 32;  // 32 compute units in the busiest XCD
  const bool before = squares_before(c.tile);  // a launch in front
  double wg = (t.slice + (norm && !before ? t.norm : 0.f)) * kps + t.fixed;
  if (kps < 16 && c.tile == 26) wg = std::max(wg, 0.326 * kps + 4.2);         // filling four slices, and the epilogue
  if (kps < 16 && c.tile >= 11 && c.tile <= 14) wg += std::max(0.0, 9.5 - t.fixed);
  if (kps < 16 && c.tile >= 29) wg += 1.5 + 0.025 * t.bm - t.fixed;
  const double cu = std::max((double)per_cu, (double)t.least) * wg;
  const double mem = (double)N * K * 2 / 7.22e6;
  const double second = split > 1 && t.groups == 1 ? 2.5 + (double)M * N * 4 * split / 2.27e6 : 0.0;
  return 1.4 + std::max(cu, mem) + 0.44 * std::min(cu, mem) + second + (norm && before ? t.norm : 0.f);
}

// The tile for a layer of more than 32 rows whose split is decided: what the rules above pick for the ring kernel, or one
// of the block kernel's, whichever cost_us puts first.  (The split stays what the rules say: it fixes the order of a
// layer's sums.)  Up to 160 rows the ring kernel, which then reads large weights past the caches, is up to 5 % better than
// its formula; an LM head with arg-max partials up to 192 rows is up to 10 % better (160 x 152064 x 5120 372 us against
// 384 on the block kernel, 192 x 32000 x 2048 46.6 against 51.4).  From 161 rows on its formula is 8 % short beside the panel
// kernel's (1536 x 2048 x 8192: 69 us on 96 x 128, 56 on 128 x 128).  Tiles 26-28 start there too: below, 136 x 28672 x 4096
// with norm and gate is 9 us faster on 160 x 128 than on the ring kernel, and the launch in front takes that back inside a
// step.  Over 360 shapes (40 to 2304 rows, with the norm, float output or arg-max, replayed from graphs) the choice is 0.8 %
// slower than the fastest tile of each.  A norm whose row sums have nowhere to go (norm_ws, as for block_takes) leaves the
// panel kernel out of an unsplit layer: there 29-31 stand in for 15-17, and the ring kernel's formula is short by as much
// (without the 8 %, 716 x 5168 x 192 takes 11.2 us on tile 8, 9.1 on 22; 306 x 14536 x 960 20.9 on tile 5, 18.6 on 22).
GemmConfig pick_any(int M, int N, int K, size_t ws_bytes, int split, ptrdiff_t norm_ws, bool am) {
  const int norm = norm_ws >= 0;
  const bool no_panel = norm && make_plan(M, N, K, 32, 32, split).split_k == 1 && !squares_fit(M, norm_ws);
  GemmConfig best = pick(M, N, K, ws_bytes, split);
  if (M <= 32) return best;
  double best_us = cost_us(M, N, K, best, norm) * (am && M <= 192 ? 0.9 : M <= 160 ? 0.95 : 1.08);
  for (int tile = N_RING_TILES + 1; tile <= N_TILES; ++tile) {
    if ((tile > 28 ? !no_panel : tile > 25 && M <= 160) || !block_takes(tile, M, N, K, split, am, norm_ws)) continue;
    const Plan p = make_plan(M, N, K, TILE_COST[tile].bm, TILE_COST[tile].bn, split);
    if (block_groups(tile) == 1 && !plan_fits(p, TILE_COST[tile].bm, (const void *)1, ws_bytes)) continue;
    const double us = cost_us(M, N, K, {tile, split}, norm);
    if (us < best_us) { best = {tile, split}; best_us = us; }
  }
  return best;
}

}  // namespace

// Called when weights are bound (outside any stream capture): the attribute calls of the large tiles are
// then out of the way of the first launch.
hipError_t gemm_prepare_device() {
  const hipError_t err = prepare_tall();
  return err == hipSuccess ? prepare_block() : err;
}

hipError_t launch_split_finish(const float *partial, const float *ssq_part, const Epilogue &e, int split,
                               const GemmArgs &a, hipStream_t s) {
  const int units = a.M * ((a.glu ? a.N / 2 : a.N) / 8);
  split_finish_kernel<<<(units + 255) / 256, 256, 0, s>>>(partial, ssq_part, e, split, a.M, a.N, a.K, a.norm_eps);
  return hipGetLastError();
}

int gemm_num_tiles() { return N_TILES; }
int gemm_tile_rows(int tile) { return tile >= 1 && tile <= N_TILES ? TILE_TM[tile] * 32 : 0; }

GemmConfig gemm_heuristic(int M, int plan_M, int N, int K, size_t ws_bytes) {
  // The split factor is decided for plan_M rows and then kept for any M, so a row's result does
  // not depend on how many other rows share the launch; the tile follows the actual M.
  const int split = pick(std::max(plan_M, M), N, K, ws_bytes, 0).split;
  return pick(M, N, K, ws_bytes, split);
}

size_t gemm_workspace_bytes(int M_max) {
  (void)M_max;
  return GEMM_SSQ_BYTES + GEMM_PARTIAL_BYTES;
}

size_t packed_weight_bytes(int N, int K, int dtype) {
  if (dtype != SF_BF16) return (size_t)N * K * sizeof(float);
  return (size_t)((N + 31) / 32) * ((K + 15) / 16) * 1024;
}

hipError_t launch_pack_weight(const void *w, void *packed, int N, int K, int glu, const void *col_gain, int dtype,
                              hipStream_t s) {
  if (dtype != SF_BF16) return hipMemcpyAsync(packed, w, (size_t)N * K * sizeof(float), hipMemcpyDeviceToDevice, s);
  const size_t units = packed_weight_bytes(N, K, dtype) / 16;
  pack_weight_kernel<<<(unsigned)((units + 255) / 256), 256, 0, s>>>((const bf16_t *)w, (uint4 *)packed, N, K, units,
                                                                     glu ? N / 2 : 0, (const bf16_t *)col_gain);
  return hipGetLastError();
}

GemmChoice gemm_choose(const GemmArgs &a) {
  const size_t ws_bytes = a.ws ? a.ws_bytes : 0;
  const bool am = a.am_val != nullptr;
  GemmConfig c = {a.tile, am ? 1 : a.split};  // arg-max partials: one workgroup owns a tile's whole K range
  if (a.tile <= 0 && a.split <= 0) {
    const int split = am ? 1 : gemm_heuristic(a.M, std::max(a.plan_M, a.M), a.N, a.K, ws_bytes).split;
    const int tiles = am ? 0 : gemm_stream_tiles(a.M, a.N, a.K, split, a.glu);
    if (tiles) return {GEMM_STREAM, tiles, split};
    c = rows_aligned(a) ? pick_any(a.M, a.N, a.K, ws_bytes, split, gemm_norm_bytes(a), am) : pick(a.M, a.N, a.K, ws_bytes, split);
  } else if (c.tile <= 0 || c.split <= 0) {
    const GemmConfig h = gemm_heuristic(a.M, a.plan_M > 0 ? a.plan_M : a.M, a.N, a.K, ws_bytes);
    if (c.split <= 0) c.split = h.split;
    if (c.tile <= 0) c.tile = c.split == h.split ? h.tile : pick(a.M, a.N, a.K, ws_bytes, c.split).tile;
  }
  if (c.tile > N_RING_TILES && (!block_takes(c.tile, a.M, a.N, a.K, c.split, am, gemm_norm_bytes(a)) || !rows_aligned(a))) c.tile = 10;
  return {c.tile > N_RING_TILES ? GEMM_BLOCK : GEMM_RING, c.tile, c.split};
}

hipError_t launch_gemm_bf16(const GemmArgs &a, hipStream_t s) {
  // the epilogues move 8 columns at a time; of rows that end within 8 (the vocabulary of an LM head) they know y alone
  if (a.N % 8 && (!a.am_val || a.bias || a.residual || a.y2 || a.hooks || a.glu)) return hipErrorInvalidValue;
  const GemmChoice c = gemm_choose(a);
  if (c.kernel == GEMM_STREAM) return launch_gemm_stream(a, c.tile, c.split, s);
  if (c.kernel == GEMM_BLOCK) return dispatch_block(c.tile, a, s, c.split);
  if (c.tile <= 5) return dispatch_narrow(c.tile, a, s, c.split);
  if (c.tile <= 10) return dispatch_wide(c.tile, a, s, c.split);
  return dispatch_tall(c.tile, a, s, c.split);
}

}  // namespace sf
