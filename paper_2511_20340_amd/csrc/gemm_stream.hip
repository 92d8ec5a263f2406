// bf16 linear layers of a handful of rows: the weights are all there is to move, and what counts is how soon every
// compute unit has its share of them in flight.
//
// The waves of a workgroup stand as KS parts of K times CG neighbouring groups of columns.  A wave streams the packed
// weight fragments of 16 or 32 columns and the few activation rows straight into registers (no LDS, no barrier in the
// loop) and multiplies with v_mfma_f32_16x16x32_bf16.  The KS partial tiles meet in LDS and are added in order of K, then
// the epilogue runs on rows of 8 columns.  So a layer whose K is split needs no second launch.
//
// The parts are those of the layer's split (make_plan), and the squares of the fused norm are summed in the ring kernel's
// order: the same bits as the ring and block kernels.
//
// 4 rows, replayed from a graph, against the ring kernel and its second launch: 2048 x 2048 8.9 -> 5.1 us, 4096 x 4096
// 11.8 -> 8.2, 6144 x 4096 13.9 -> 10.5, 2048 x 8192 12.1 -> 10.4, 4096 x 14336 23.8 -> 19.8, 16384 x 2048 (unsplit)
// 15.6 -> 13.3.
#include "gemm_common.h"

#include <algorithm>

namespace sf {
namespace {

// waves side by side: four waves to a workgroup at least
constexpr int stream_groups(int KS) { return KS >= 4 ? 1 : 4 / KS; }
// 32-position chunks of K per batch, two batches in flight: bounded by the registers of 16 waves a compute unit, of 8
// where a workgroup has but four; even, so that a chunk's place in its 64-position slice is known
constexpr int stream_batch(int TM, int TN, int KS) {
  const int regs = KS <= 4 ? 16 : 8;
  return regs / (TM + TN) / 2 * 2;
}

// TM: 16-row tiles of activations, TN: 16-column tiles of weights per wave; NORM: the rows are to be RMS-normalised (the
// gains are folded into the weights, the row factor is formed here); ONCE: non-temporal weight loads
template <int TM, int TN, int KS, int NORM, int ONCE>
__global__ __launch_bounds__(64 * KS * stream_groups(KS), KS <= 4 ? 2 : 4) void gemm_stream_kernel(
    const bf16_t *__restrict__ A, const uint4 *__restrict__ Wp, const Epilogue e, int M, int N, int K, int chunks_per_part,
    float eps) {
  constexpr int CG = stream_groups(KS), U = stream_batch(TM, TN, KS), THREADS = 64 * KS * CG;
  constexpr int TILE = TM * TN * 256, COLS = 16 * TN * CG;
  __shared__ __attribute__((aligned(16))) float part[KS * CG * TILE];
  __shared__ float sq[KS][16 * TM];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / CG, cg = wave % CG;
  const int r = lane & 15, kg = lane >> 4;
  const int k_steps = (K + 15) >> 4, chunks = (K + 31) >> 5;
  const int c0 = ks * chunks_per_part, c1 = min(c0 + chunks_per_part, chunks);
  const int whole = min(c1, K >> 5);  // the chunks before this one lie inside K
  const int m0 = blockIdx.y * 16 * TM, n0 = blockIdx.x * COLS;

  const bf16_t *ap[TM];
#pragma unroll
  for (int a = 0; a < TM; ++a) ap[a] = A + (size_t)min(m0 + a * 16 + r, M - 1) * K;
  // column tile b: rows n % 32 .. +15 of packed row block n / 32 (the last block again past the end); a lane's 8 positions
  // sit in unit 2 c + kg / 2 of chunk c, half kg % 2
  const uint4 *wp[TN];
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int n = n0 + (cg * TN + b) * 16, block = min(n >> 5, ((N + 31) >> 5) - 1);
    wp[b] = Wp + (size_t)block * k_steps * 64 + (kg & 1) * 32 + (n & 16) + r;
  }

  f32x4 acc[TM][TN];
  float ssq[2][TM];  // of the chunks with an even and an odd number
#pragma unroll
  for (int a = 0; a < TM; ++a) {
    ssq[0][a] = ssq[1][a] = 0.f;
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  uint4 wf[2][U][TN], af[2][U][TM];
  // loads are unconditional, so that the compiler can count how many are in flight; chunks past the part repeat its last
  auto load = [&](int buf, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int unit = min(2 * min(c + u, c1 - 1) + (kg >> 1), k_steps - 1);
#pragma unroll
      for (int b = 0; b < TN; ++b) wf[buf][u][b] = load_unit<ONCE>(wp[b] + (size_t)unit * 64);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int a = 0; a < TM; ++a)
        af[buf][u][a] = *reinterpret_cast<const uint4 *>(ap[a] + min(min(c + u, c1 - 1) * 32 + kg * 8, K - 8));
  };
  auto product = [&](int odd, const uint4 (&va)[TM], const uint4 (&vw)[TN]) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const uint4 v = va[a];
      if (NORM) {
        float t = ssq[odd][a];
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.x), __builtin_bit_cast(bf16x2, v.x), t, false);
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.y), __builtin_bit_cast(bf16x2, v.y), t, false);
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.z), __builtin_bit_cast(bf16x2, v.z), t, false);
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.w), __builtin_bit_cast(bf16x2, v.w), t, false);
        ssq[odd][a] = t;
      }
#pragma unroll
      for (int b = 0; b < TN; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, vw[b]),
                                                            acc[a][b], 0, 0, 0);
    }
  };
  auto multiply = [&](int buf, int c) __attribute__((always_inline)) {
    if (c + U <= whole) {
#pragma unroll
      for (int u = 0; u < U; ++u) product(u & 1, af[buf][u], wf[buf][u]);
      return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c + u >= c1) continue;
      // both operands are zero past K: a zero times what the clamped address holds need not be zero
      const bool in = (c + u) * 32 + kg * 8 < K;
      uint4 va[TM], vw[TN];
#pragma unroll
      for (int a = 0; a < TM; ++a) va[a] = in ? af[buf][u][a] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int b = 0; b < TN; ++b) vw[b] = in ? wf[buf][u][b] : make_uint4(0, 0, 0, 0);
      product(u & 1, va, vw);
    }
  };
  if (c0 < c1) {
    load(0, c0);
    for (int c = c0; c < c1; c += 2 * U) {
      load(1, c + U);
      __builtin_amdgcn_sched_barrier(0);  // a batch is requested whole before the one ahead of it is multiplied
      multiply(0, c);
      load(0, c + 2 * U);
      __builtin_amdgcn_sched_barrier(0);
      multiply(1, c + U);
    }
  }

#pragma unroll
  for (int a = 0; a < TM; ++a) {
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[wave * TILE + (a * TN + b) * 256 + (kg * 4 + v) * 16 + r] = acc[a][b][v];
    if (NORM) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        ssq[h][a] += __shfl_xor(ssq[h][a], 16);
        ssq[h][a] += __shfl_xor(ssq[h][a], 32);
      }
      if (cg == 0 && kg == 0) sq[ks][a * 16 + r] = ssq[0][a] + ssq[1][a];
    }
  }
  __syncthreads();
  // one thread per row and 8 columns (with the gate: 8 features, columns f and f + 16 of a pair of tiles)
  const int groups = e.glu ? COLS / 16 : COLS / 8;
  for (int item = tid; item < 16 * TM * groups; item += THREADS) {
    const int row = item / groups, g = item - row * groups, a = row >> 4;
    const int c8 = e.glu ? (g >> 1) * 32 + (g & 1) * 8 : g * 8;
    if (m0 + row >= M) return;
    auto total = [&](int col, float (&v)[8]) __attribute__((always_inline)) {
      const int tile = col >> 4;
      const float *p = part + tile / TN * TILE + (a * TN + tile % TN) * 256 + (row & 15) * 16 + (col & 15);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4 q = *reinterpret_cast<const f32x4 *>(p + s * CG * TILE + j * 4);
#pragma unroll
          for (int i = 0; i < 4; ++i) v[j * 4 + i] += q[i];
        }
    };
    float rinv = 1.f;
    if (NORM) {
      float t = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) t += sq[s][row];
      rinv = 1.0f / sqrtf(t / (float)K + eps);
    }
    float v[8];
    total(c8, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= rinv;
    if (e.glu) {
      const int f = (n0 >> 1) + g * 8;
      float up[8];
      total(c8 + 16, up);
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = v[i] / (1.0f + __expf(-v[i])) * (up[i] * rinv);
      if (f < (N >> 1)) store_n(reinterpret_cast<bf16_t *>(e.y) + (size_t)(m0 + row) * (N >> 1) + f, v, e.vec);
      continue;
    }
    const int col = n0 + c8;
    if (col < N) finish_row8(e, m0 + row, col, N, v);
  }
}

template <int TM, int TN, int KS>
hipError_t run(const GemmArgs &a, hipStream_t s) {
  constexpr int COLS = 16 * TN * stream_groups(KS);
  if (a.am_val || (a.glu && COLS % 32)) return hipErrorInvalidValue;
  const Epilogue e = make_epilogue(a);
  const dim3 grid((a.N + COLS - 1) / COLS, (a.M + 16 * TM - 1) / (16 * TM));
  const Plan p = make_plan(a.M, a.N, a.K, 16 * TM, COLS, KS);
  auto launch = [&](auto kernel) {
    kernel<<<grid, 64 * KS * stream_groups(KS), 0, s>>>((const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N, a.K,
                                                        p.kt_per_split * (BK / 32), a.norm_eps);
  };
  if (weights_once(a, grid.y)) launch(a.fused_norm ? &gemm_stream_kernel<TM, TN, KS, 1, 1> : &gemm_stream_kernel<TM, TN, KS, 0, 1>);
  else launch(a.fused_norm ? &gemm_stream_kernel<TM, TN, KS, 1, 0> : &gemm_stream_kernel<TM, TN, KS, 0, 0>);
  return hipGetLastError();
}
template <int TM, int TN>
hipError_t run(const GemmArgs &a, int split, hipStream_t s) {
  switch (split) {
    case 1: return run<TM, TN, 1>(a, s);
    case 2: return run<TM, TN, 2>(a, s);
    case 4: return run<TM, TN, 4>(a, s);
    case 8: return run<TM, TN, 8>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// What a launch takes, in us, fitted to 1800 measured ones (1 to 32 rows, 64 to 28672 columns, K 512 to 24576, splits 1 to
// 8, weights cold, replayed from a graph): the streaming kernel 8.2 % rms, the ring kernel on its 32-row tile 6.9 %.  A
// compute unit takes in rows and columns of its share of K, workgroup after workgroup; the weights have to come from
// memory; the ring kernel pays for the second launch of a split.
static double stream_us(int M, int N, int K, int split, int tiles) {
  const int groups = stream_groups(split), cols = 16 * tiles * groups;
  const int rounds = ((N + cols - 1) / cols * ((M + 31) / 32) + 255) / 256;
  const double cu = rounds * ((22.8 * M + 11.6 * 16 * tiles + 68.6) * K * groups * 2e-6 + 0.73), mem = N * (2.0 * K) / 8.76e6;
  return 2.0 + std::max(cu, mem) + 0.52 * std::min(cu, mem);
}
static double ring_us(int M, int N, int K, int split) {
  const int KT = (K + BK - 1) / BK, slices = (KT + split - 1) / split, wgs = (N + 127) / 128 * split;
  const double cu = std::max((double)((wgs + 255) / 256), 1.78) * (0.045 * slices + 2.66), mem = N * (2.0 * K) / 8.07e6;
  return std::max(cu, mem) + 0.96 * std::min(cu, mem) + (split > 1 ? 2.79 + 0.93e-6 * M * N * 4.0 * split : 0.0);
}

// Up to 32 rows the formulas decide; over the measured shapes the choice is 0.5 % slower than the fastest kernel of each.
// Every workgroup reads all rows, so they have to stay few beside its 16 or 32 weight rows, and few columns under a long K
// keep few compute units busy: 32 x 4096 x 4096 takes 13.8 us on the ring kernel and 13.0 here, 32 x 2048 x 8192 14.1 and
// 21.7, 32 x 512 x 24576 17 and 52.
// More rows: every 32 of them read the weights again.  That pays only where the ring kernel would need its second launch
// (splits of 4, which the block kernel's groups of waves take at fewer shapes, and K of no whole slices, which it never
// takes), all workgroups run at once and the rows' share of a compute unit's intake stays small: 64 x 512 x 2048 9.6 -> 7.2
// us, 64 x 2048 x 2048 10.6 -> 8.1, 96 x 512 x 1000 9.1 -> 5.7; with K = 4096 it would be 12.0 -> 11.4 and 15.1 -> 14.8.
int gemm_stream_tiles(int M, int N, int K, int split, int glu) {
  if (split != 1 && split != 2 && split != 4 && split != 8) return 0;
  const int groups = stream_groups(split);
  if (M > 32) {
    const int row_tiles = (M + 31) / 32;
    const int tiles = (glu && groups == 1) || (long)((N + 16 * groups - 1) / (16 * groups)) * row_tiles > 256 ? 2 : 1;
    const int cols = 16 * tiles * groups;
    const bool second_launch = split == 4 || split == 8 || (split == 2 && K % BK);
    return second_launch && (long)K * groups <= 2048 && (long)((N + cols - 1) / cols) * row_tiles <= 256 ? tiles : 0;
  }
  int best = 0;
  double best_us = ring_us(M, N, K, split);
  for (int tiles = 1; tiles <= 2; ++tiles) {
    if (glu && groups * tiles % 2) continue;
    const double us = stream_us(M, N, K, split, tiles);
    if (us < best_us) { best = tiles; best_us = us; }
  }
  return best;
}

hipError_t launch_gemm_stream(const GemmArgs &a, int tiles, int split, hipStream_t s) {
  if (a.M <= 16) return tiles == 2 ? run<1, 2>(a, split, s) : run<1, 1>(a, split, s);
  return tiles == 2 ? run<2, 2>(a, split, s) : run<2, 1>(a, split, s);
}

}  // namespace sf
