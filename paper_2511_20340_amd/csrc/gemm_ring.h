// Linear layers  y[M][N] = x[M][K] . w[N][K]^T (+bias) (+residual)  for gfx950.
//
// bf16 path ("weight-direct").  Decoding GEMMs are skinny: M = B*(k+1) rows against weight
// matrices that are streamed from HBM exactly once.  The weights are therefore kept PACKED in
// MFMA-operand order (pack_weight below): for every 32-row block of W and every 16-wide k-step
// one 1 KiB unit holds, lane by lane, the 8 bf16 a lane feeds to v_mfma_f32_32x32x16_bf16.  A
// wavefront owns one such row block per output tile and streams its units straight from global
// memory into operand registers with fully coalesced 16-byte loads -- no LDS traffic, no barrier
// on the weight side.  Only the activations (BM = TM*32 rows x 64 k) are staged through LDS
// (double buffer, rows padded to 72 elements: conflict-free 16-byte operand reads) and shared by
// the 4 or 8 waves of the workgroup, which cover 128 or 256 output columns.
//
// Memory pipeline: every wave keeps a ring of R K-slices in flight (weights in registers, the
// activation chunks that go with them in registers until their turn to enter LDS).  All loads are
// unconditional and issued in the order of use, so the compiler's vmcnt waits only ever cover the
// slice that is needed next.
//
// Parallelism for small N*M: the K dimension is split over `split_k` workgroups per tile.  Each leaves its fp32
// partial tile in the workspace; a second, elementwise launch (split_finish_kernel) adds the partials in split
// order (deterministic) and applies the epilogue with the whole chip.
//
// Workgroup ids are remapped so that all M-tiles of one weight column block (and K split) run on the
// same XCD (its L2 then serves the weight units to every M-tile after one HBM read), and those units are
// dealt evenly over the eight XCDs.
//
// The kernel lives in this header; gemm_tiles_*.hip instantiate it for the tile configurations, gemm.hip chooses among
// them.
#pragma once
#include "gemm_common.h"

#include <cstdint>
#include <type_traits>
#include <utility>

namespace sf {
namespace {

// f(integral_constant<0>) ... f(integral_constant<N-1>): a loop whose index is a compile-time constant in
// every iteration
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// max over the 32 lanes that share (lane >> 5): quad permutes, the two row mirrors, one cross-row exchange.
// maxNum semantics: a NaN operand is ignored.
__device__ __forceinline__ float half_wave_max(float v) {
#define SF_DPP(x, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, false))
  v = fmaxf(v, SF_DPP(v, 0xB1));   // quad_perm [1,0,3,2]
  v = fmaxf(v, SF_DPP(v, 0x4E));   // quad_perm [2,3,0,1]
  v = fmaxf(v, SF_DPP(v, 0x141));  // row_half_mirror: quads of an 8-lane group
  v = fmaxf(v, SF_DPP(v, 0x140));  // row_mirror: the two 8-lane groups of a 16-lane row
#undef SF_DPP
  return fmaxf(v, __shfl_xor(v, 16));
}

// Row length (floats) of the LDS piece a wave turns a 32x32 tile in: rows stay 16-byte aligned, and the two rows
// four apart that one store instruction writes land in different halves of the 64 banks.
constexpr int TURN_STRIDE = 40;

// What every bf16 kernel variant does once a workgroup holds its accumulators.
//
// Fused RMSNorm (sS != nullptr): the weight was packed with the norm's gain vector folded into its
// columns, the main loop ran on the raw activations and left each row's sum of squares over this
// workgroup's K range in sS[BM]; the row factor 1/sqrt(mean(x^2)+eps) commutes with the K sum and
// is applied to the finished tiles here.
//
// Split K (split_k > 1): partial tile and row sums go to the workspace as rows of [split][M][N] and [split][M], and
// split_finish_kernel does the rest.
//
// The NW waves stand in WM rows of NW / WM; a wave holds TM x TN tiles, block row (wave / (NW / WM)) * TM first.
// nb0: the wave's first 32-column block.
//
// scratch: LDS the main loop no longer needs, at least NW * TM * 32 * 8 (arg-max partials) and NW * 128 * TURN_STRIDE bytes.
template <int TM, int TN, int NW = 4, int WM = 1>
__device__ __forceinline__ void gemm_finish(f32x16 (&acc)[TM][TN], const Epilogue &e, int M, int N, int split_k,
                                            float *__restrict__ partial, int tn, int ks, int m0, int nb0,
                                            void *scratch, float *sS = nullptr, float *__restrict__ ssq_part = nullptr,
                                            int K = 1, float eps = 0.f) {
  constexpr int BM = WM * TM * 32, WN = NW / WM;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ln = lane & 31, lh = lane >> 5;
  const int a_w = WM == 1 ? 0 : wave / WN * TM;  // this wave's first 32-row block

  // A lane holds one column of 16 rows of every 32x32 tile; stored from there, an element is a 2- or 4-byte store
  // of its own, and those stores cost more than the K loop of a short layer (160 x 2048 x 512 on 160-row tiles:
  // 20.1 us, 11.1 us this way).  So each wave turns its tiles through a private piece of LDS, one after the other, and
  // a lane then holds 16 / W groups of W consecutive columns: W = 4 where floats are stored (eight lanes a row, so one
  // instruction writes whole 128-byte lines of 8 rows; with two groups of 8 columns a lane every line is left to four
  // instructions: 4096 x 16384 x 2048 with a float output 282 us, 342 that way), W = 8 where bf16 is (four lanes a row).
  // The two rows that a quarter of a wave reads are four apart: different halves of the banks, as for the writes.
  float *turn = reinterpret_cast<float *>(scratch) + wave * (32 * TURN_STRIDE);
  auto unit_row = [&](int W, int u) __attribute__((always_inline)) {
    return W == 4 ? u * 8 + (lane >> 3 & 1) * 4 + (lane >> 4) : u * 16 + (lane >> 2);
  };
  auto unit_col = [&](int W) __attribute__((always_inline)) { return W == 4 ? (lane & 7) * 4 : (lane & 3) * 8; };
  auto put = [&](const f32x16 &c) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);  // tile by tile: overlapping them would cost registers the tall tiles lack
#pragma unroll
    for (int i = 0; i < 16; ++i) turn[c_row(i, lh) * TURN_STRIDE + ln] = c[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto taken = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto transpose = [&](auto w_c, const f32x16 &c, float (&v)[16]) __attribute__((always_inline)) {
    constexpr int W = decltype(w_c)::value;
    put(c);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 q = *reinterpret_cast<const f32x4 *>(turn + unit_row(W, j / (W / 4)) * TURN_STRIDE + unit_col(W) + j % (W / 4) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j * 4 + i] = q[i];
    }
    taken();
  };

  if (split_k > 1) {
    if (sS && tn == 0 && tid < BM && m0 + tid < M) ssq_part[(size_t)ks * M + m0 + tid] = sS[tid];
    __syncthreads();  // the other waves are done with the LDS this one is about to write
    static_for<TM * TN>([&](auto i_c) {
      constexpr int a = decltype(i_c)::value / TN, b = decltype(i_c)::value % TN;
      float v[16];
      transpose(std::integral_constant<int, 4>{}, acc[a][b], v);
      const int col = (nb0 + b) * 32 + unit_col(4);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int row = m0 + (a_w + a) * 32 + unit_row(4, u);
        if (row < M && col < N)
          store_n(partial + ((size_t)ks * M + row) * N + col, reinterpret_cast<const float(&)[4]>(v[u * 4]), 1);
      }
    });
    return;
  }

  if (sS && tid < BM) sS[tid] = 1.0f / sqrtf(sS[tid] / (float)K + eps);  // one row factor per row, once

  if (e.am_val) {
    // Arg-max partials of this workgroup's column tile: per row the largest accumulator and the lowest
    // column that holds it.  Columns past N and NaN never take part.
    float *s_val = reinterpret_cast<float *>(scratch);       // [WN][BM]
    int32_t *s_idx = reinterpret_cast<int32_t *>(s_val + WN * BM);
    const int w_n = WM == 1 ? wave : wave % WN;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float best_v = -__builtin_huge_valf();
        int32_t best_i = INT32_MAX;
#pragma unroll
        for (int b = 0; b < TN; ++b) {
          const int col = (nb0 + b) * 32 + ln;
          const float x = col < N ? acc[a][b][v] : -__builtin_huge_valf();
          const float mx = half_wave_max(x);
          const unsigned long long bal = __ballot(col < N && x == mx);
          const uint32_t half = lh ? (uint32_t)(bal >> 32) : (uint32_t)bal;
          if (half != 0 && mx > best_v) {  // later blocks hold higher columns: strictly greater only
            best_v = mx;
            best_i = (nb0 + b) * 32 + (__ffs(half) - 1);
          } else if (half != 0 && best_i == INT32_MAX) {  // a tile of -inf only: its first column
            best_v = mx;
            best_i = (nb0 + b) * 32 + (__ffs(half) - 1);
          }
        }
        if (ln == 0) {
          s_val[w_n * BM + (a_w + a) * 32 + c_row(v, lh)] = best_v;
          s_idx[w_n * BM + (a_w + a) * 32 + c_row(v, lh)] = best_i;
        }
      }
    __syncthreads();
    if (tid < BM && m0 + tid < M) {
      float bv = s_val[tid];
      int32_t bi = s_idx[tid];
#pragma unroll
      for (int w = 1; w < WN; ++w) {  // waves hold ascending column ranges
        const float v = s_val[w * BM + tid];
        const int32_t i = s_idx[w * BM + tid];
        if (i != INT32_MAX && (bi == INT32_MAX || v > bv)) { bv = v; bi = i; }
      }
      e.am_val[(size_t)(m0 + tid) * e.am_stride + tn] = bv;
      e.am_idx[(size_t)(m0 + tid) * e.am_stride + tn] = bi;
    }
    if (!e.y) return;
  }

  __syncthreads();  // row factors are in place; the other waves are done with the LDS this one is about to write
  if (e.glu) {
    // SwiGLU.  The weight was packed with gate and up rows interleaved 16 by 16: columns 0-15 of a tile are gate
    // features f..f+15, columns 16-31 the matching up features.  Lane l takes 8 features of both.
    const int F = N >> 1;
    const int t_row = lane >> 1, t_col = (lane & 1) * 8;
    static_for<TM * TN>([&](auto i_c) {
      constexpr int a = decltype(i_c)::value / TN, b = decltype(i_c)::value % TN;
      const int col = (nb0 + b) * 16 + t_col, row = m0 + (a_w + a) * 32 + t_row;
      float v[16];
      put(acc[a][b]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 q = *reinterpret_cast<const f32x4 *>(turn + t_row * TURN_STRIDE + t_col + (j >> 1) * 16 + (j & 1) * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[j * 4 + i] = q[i];
      }
      taken();
      if (sS) {
        const float f = sS[(a_w + a) * 32 + t_row];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] *= f;
      }
      float r[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = v[i] / (1.0f + __expf(-v[i])) * v[8 + i];
      if (row < M && col < F) store_n(reinterpret_cast<bf16_t *>(e.y) + (size_t)row * F + col, r, e.vec);
    });
    return;
  }

  // The residual values of a group of tiles are requested before the group's first store (y may be the residual
  // buffer itself): one exposed round trip per group.  A wave with up to five tiles forms one group, taller ones
  // go five, the tallest (no registers to spare) two tiles at a time.
  // constant tile indices whatever the size of the body: an unroll pragma gives up beyond a size threshold, and a
  // run-time index into the accumulators would move them out of registers
  constexpr int MOST = TM * TN > 7 ? 2 : 5;  // tiles per group
  constexpr int AG = TN >= MOST ? 1 : (TM < MOST / TN ? TM : MOST / TN), GROUPS = (TM + AG - 1) / AG;
  auto store_all = [&](auto w_c) __attribute__((always_inline)) {
    constexpr int W = decltype(w_c)::value, UNITS = 16 / W;
    auto load_residual = [&](int a, int b, float (&res)[16]) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        const int row = min(m0 + (a_w + a) * 32 + unit_row(W, u), M - 1);
        const size_t o = (size_t)row * N + min((nb0 + b) * 32 + unit_col(W), N - W);
        float(&dst)[W] = reinterpret_cast<float(&)[W]>(res[u * W]);
        if (e.res_f32) load_n(reinterpret_cast<const float *>(e.residual) + o, dst, e.vec);
        else load_n(reinterpret_cast<const bf16_t *>(e.residual) + o, dst, e.vec);
      }
    };
    auto store_tile = [&](int a, int b, const f32x16 &c, const float (&res)[16]) __attribute__((always_inline)) {
      float v[16];
      transpose(w_c, c, v);
      const int col = (nb0 + b) * 32 + unit_col(W);
      float bv[W];
      if (e.bias) load_n(e.bias + min(col, N - W), bv, e.vec);
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        const int in_tile = (a_w + a) * 32 + unit_row(W, u), row = m0 + in_tile;
        if (row >= M || col >= N) continue;
        const float f = sS ? sS[in_tile] : 1.f;
        float r[W];
#pragma unroll
        for (int i = 0; i < W; ++i) {
          r[i] = sS ? v[u * W + i] * f : v[u * W + i];
          if (e.bias) r[i] += bv[i];
          if (e.residual) r[i] += res[u * W + i];
        }
        store_row(e, row, col, N, r);
      }
    };
    static_for<GROUPS>([&](auto g_c) {
      constexpr int a0 = decltype(g_c)::value * AG, a1 = a0 + AG < TM ? a0 + AG : TM;
      float res[AG][TN][16];
      if (e.residual) {
#pragma unroll
        for (int a = a0; a < a1; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) load_residual(a, b, res[a - a0][b]);
      }
#pragma unroll
      for (int a = a0; a < a1; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) store_tile(a, b, acc[a][b], res[a - a0][b]);
    });
  };
  if (e.out_f32) store_all(std::integral_constant<int, 4>{});
  else store_all(std::integral_constant<int, 8>{});
}

// Dynamic LDS of a workgroup: the activation double buffer, later the epilogue's transposition pieces (+ the fused
// norm's row sums behind them).
template <int TM, int NW>
constexpr size_t lds_loop_bytes() {
  constexpr size_t loop = (size_t)2 * TM * 32 * LDK * sizeof(bf16_t), turn = (size_t)NW * 32 * TURN_STRIDE * sizeof(float);
  return loop > turn ? loop : turn;
}
template <int TM, int NW>
constexpr size_t lds_bytes(bool norm) {
  return lds_loop_bytes<TM, NW>() + (norm ? (size_t)TM * 32 * sizeof(float) : 0);
}

// The bf16 kernel.  TM 32-row activation blocks x TN weight row blocks per wave, NW waves, ring
// depth R.  Slot indices are compile-time after unrolling by R; the loop runs whole rounds of R
// slices, and slices past the workgroup's K range contribute zeros.
template <int TM, int TN, int R, int OCC, int NW, int NORM, int PIPE, int ONCE>
__global__ __launch_bounds__(64 * NW, OCC) void gemm_ring_kernel(const bf16_t *__restrict__ A,
                                                        const uint4 *__restrict__ Wp, const Epilogue e, int M,
                                                        int N, int K, int tiles_m, int tiles_n, int split_k,
                                                        int kt_per_split, float *__restrict__ partial, float eps,
                                                        float *__restrict__ ssq_part) {
  static_assert(R >= 2, "the slot after the current one holds the next activation chunk");
  constexpr int BM = TM * 32;
  constexpr int NT = 64 * NW;              // threads
  constexpr int CH = TM * 256;             // 16-byte activation chunks per K slice
  constexpr int CPT = (CH + NT - 1) / NT;  // chunks per thread
  // [2][BM][LDK] activations (later the transposition pieces); NORM: then float sS[BM], the rows' sums of squares
  extern __shared__ __attribute__((aligned(16))) bf16_t sA[];

  // Consecutive workgroup ids go to consecutive XCDs.  The M-tiles of one (column tile, K split) unit read
  // the same weight bytes: they get consecutive slots of ONE XCD, and the units are dealt round-robin over
  // the XCDs, so no XCD holds more than one unit above the average.
  const int id = blockIdx.x;
  const int xcd = id % XCDS, j = id / XCDS;
  const int tm = j % tiles_m, unit = (j / tiles_m) * XCDS + xcd;
  if (unit >= tiles_n * split_k) return;
  const int tn = unit / split_k, ks = unit % split_k;
  const int m0 = tm * BM;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ln = lane & 31, lh = lane >> 5;
  const int n_blocks = (N + 31) >> 5;
  const int k_steps = (K + 15) >> 4;
  const int nb0 = (tn * NW + wave) * TN;
  const int KT = (K + BK - 1) / BK;
  const int kt0 = ks * kt_per_split, kt1 = min(KT, kt0 + kt_per_split);
  float *sS = reinterpret_cast<float *>(reinterpret_cast<char *>(sA) + lds_loop_bytes<TM, NW>());
  float ssq[CPT];
#pragma unroll
  for (int c = 0; c < CPT; ++c) ssq[c] = 0.f;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  uint4 ra[R][CPT];
  uint4 w[R][4][TN];
  // Every load is unconditional (addresses clamped into the operands), so the compiler can count
  // how many are in flight.  Rows >= M and columns >= N compute garbage that the epilogue never
  // writes; K positions outside this workgroup's slice are zeroed on the activation side when the
  // chunk goes to LDS, which silences whatever weight the clamped address fetched.
  auto aload = [&](uint4 (&r)[CPT], int kt) {
    const int ktc = min(kt, KT - 1);
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int cid = min(tid + NT * c, CH - 1), row = cid >> 3, kc = (cid & 7) * 8;
      const int gr = min(m0 + row, M - 1), kk = min(ktc * BK + kc, K - 8);
      r[c] = *reinterpret_cast<const uint4 *>(A + (size_t)gr * K + kk);
    }
  };
  auto astore = [&](int buf, const uint4 (&r)[CPT], int kt) {
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      const int cid = tid + NT * c, row = cid >> 3, kc = (cid & 7) * 8;
      if (CH % NT != 0 && cid >= CH) continue;
      const bool live = kt < kt1 && kt * BK + kc < K;
      uint4 v = r[c];
      v.x = live ? v.x : 0u; v.y = live ? v.y : 0u; v.z = live ? v.z : 0u; v.w = live ? v.w : 0u;
      if (NORM) {  // the row's sum of squares, two bf16 products per instruction
        float t = ssq[c];
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.x), __builtin_bit_cast(bf16x2, v.x), t, false);
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.y), __builtin_bit_cast(bf16x2, v.y), t, false);
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.z), __builtin_bit_cast(bf16x2, v.z), t, false);
        t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.w), __builtin_bit_cast(bf16x2, v.w), t, false);
        ssq[c] = t;
      }
      *reinterpret_cast<uint4 *>(sA + (buf * BM + row) * LDK + kc) = v;
    }
  };
  auto wload = [&](uint4 (&wr)[4][TN], int kt) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int b = 0; b < TN; ++b) {
        const int kstep = min(kt * 4 + s, k_steps - 1), nb = min(nb0 + b, n_blocks - 1);
        wr[s][b] = load_unit<ONCE>(Wp + ((size_t)nb * k_steps + kstep) * 64 + lane);
      }
  };

#pragma unroll
  for (int r = 0; r < R; ++r) {
    aload(ra[r], kt0 + r);
    wload(w[r], kt0 + r);
  }
  astore(0, ra[0], kt0);
  __syncthreads();
  for (int base = kt0; base < kt1; base += R) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int kt = base + r, buf = (kt - kt0) & 1;
      const bf16_t *pa = sA + (buf * BM + ln) * LDK + lh * 8;
      // The three issue orders below are written out in full: sharing their pieces through helpers changes the
      // register allocation and the schedule of every variant, and each was measured as it stands.
      if constexpr (PIPE == 2) {
        // Light pinning for tiles without the registers for the order below: each k-step's weight registers
        // are refilled right after its products, the next slice's chunk goes to LDS after k-step 1, the
        // slot's next activation chunk is requested after k-step 2; fragments are read where they are used.
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
          for (int a = 0; a < TM; ++a) {
            const bf16x8 f =
                __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + a * 32 * LDK + s * 16));
#pragma unroll
            for (int b = 0; b < TN; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, __builtin_bit_cast(bf16x8, w[r][s][b]),
                                                                  acc[a][b], 0, 0, 0);
          }
          if (s == 1) astore(buf ^ 1, ra[(r + 1) % R], kt + 1);
          if (s == 2) aload(ra[r], kt + R);
#pragma unroll
          for (int b = 0; b < TN; ++b) {
            const int kstep = min((kt + R) * 4 + s, k_steps - 1), nb = min(nb0 + b, n_blocks - 1);
            w[r][s][b] = load_unit<ONCE>(Wp + ((size_t)nb * k_steps + kstep) * 64 + lane);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        continue;
      }
      if constexpr (PIPE == 1) {
        // Issue order pinned by hand: the slot's next activation chunk is requested first; the activation
        // fragments of k-step s + 1 are requested before the products of k-step s are issued, so that the LDS
        // latency of all but the slice's first k-step runs under MFMAs; each k-step's weight registers are
        // refilled as soon as its products are issued.
        bf16x8 fa[2][TM];
#pragma unroll
        for (int a = 0; a < TM; ++a)
          fa[0][a] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + a * 32 * LDK));
        aload(ra[r], kt + R);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          if (s + 1 < 4) {
#pragma unroll
            for (int a = 0; a < TM; ++a)
              fa[(s + 1) & 1][a] =
                  __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + a * 32 * LDK + (s + 1) * 16));
          }
          if (s == 1) astore(buf ^ 1, ra[(r + 1) % R], kt + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s & 1][a], __builtin_bit_cast(bf16x8, w[r][s][b]),
                                                                  acc[a][b], 0, 0, 0);
#pragma unroll
          for (int b = 0; b < TN; ++b) {
            const int kstep = min((kt + R) * 4 + s, k_steps - 1), nb = min(nb0 + b, n_blocks - 1);
            w[r][s][b] = load_unit<ONCE>(Wp + ((size_t)nb * k_steps + kstep) * 64 + lane);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        continue;
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int a = 0; a < TM; ++a) {
          const bf16x8 fa =
              __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(pa + a * 32 * LDK + s * 16));
#pragma unroll
          for (int b = 0; b < TN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, __builtin_bit_cast(bf16x8, w[r][s][b]),
                                                                acc[a][b], 0, 0, 0);
        }
      }
      astore(buf ^ 1, ra[(r + 1) % R], kt + 1);  // the chunk of slice kt + 1
      aload(ra[r], kt + R);              // this slot's next tenant, activations first: needed first
      wload(w[r], kt + R);
      __syncthreads();
    }
  }
  if (NORM) {
    // the 8 threads that carried a row's chunks sit in adjacent lanes
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
      float t = ssq[c];
      t += __shfl_xor(t, 1);
      t += __shfl_xor(t, 2);
      t += __shfl_xor(t, 4);
      const int cid = tid + NT * c;
      if ((tid & 7) == 0 && cid < CH) sS[cid >> 3] = t;
    }
    __syncthreads();
  }
  gemm_finish<TM, TN, NW>(acc, e, M, N, split_k, partial, tn, ks, m0, nb0, sA, NORM ? sS : nullptr, ssq_part, K, eps);
}

// A tile whose activation double buffer exceeds the 64 KiB of dynamic LDS a kernel gets by default has the
// limit of both its kernels (with and without the fused norm) raised, once per device.
template <int TM, int TN, int R, int OCC, int NW, int PIPE = 0, int PIPE_NORM = PIPE>
hipError_t ensure_lds() {
  constexpr int cap = (int)lds_bytes<TM, NW>(true);
  if (cap <= 64 * 1024) return hipSuccess;
  static bool raised[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (raised[dev]) return hipSuccess;
  auto raise = [](const void *f) { return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, cap); };
  hipError_t err = raise(reinterpret_cast<const void *>(&gemm_ring_kernel<TM, TN, R, OCC, NW, 1, PIPE_NORM, 0>));
  if (err == hipSuccess) err = raise(reinterpret_cast<const void *>(&gemm_ring_kernel<TM, TN, R, OCC, NW, 0, PIPE, 0>));
  if (err == hipSuccess) raised[dev] = true;
  return err;
}

// PIPE: issue order of the plain kernel, PIPE_NORM: of the one with the fused norm
template <int TM, int TN, int R, int OCC, int NW, int PIPE = 0, int PIPE_NORM = PIPE>
hipError_t run_ring(const GemmArgs &a, hipStream_t s, int split) {
  constexpr int BM = TM * 32, BN = NW * TN * 32;
  const Plan p = make_plan(a.M, a.N, a.K, BM, BN, split);
  if (!plan_fits(p, BM, a.ws, a.ws_bytes)) return hipErrorInvalidValue;
  const int groups = (p.tiles_n * p.split_k + XCDS - 1) / XCDS;  // (column tile, K split) units per XCD
  const size_t lds = lds_bytes<TM, NW>(a.fused_norm != 0);
  float *ssq_part = p.split_k > 1 ? (float *)a.ws : nullptr;
  float *partial = p.split_k > 1 ? (float *)((char *)a.ws + GEMM_SSQ_BYTES) : nullptr;
  const dim3 grid(groups * XCDS * p.tiles_m), block(64 * NW);
  if (a.am_val && (p.split_k != 1 || a.am_stride < p.tiles_n || a.fused_norm)) return hipErrorInvalidValue;
  if (a.am_val && a.am_parts_out) *a.am_parts_out = p.tiles_n;
  static_assert((size_t)2 * BM * LDK * sizeof(bf16_t) >= (size_t)NW * BM * 8, "arg-max partials fit the activation tile");
  const Epilogue e = make_epilogue(a);
  if (lds > 64 * 1024) {
    const hipError_t err = ensure_lds<TM, TN, R, OCC, NW, PIPE, PIPE_NORM>();
    if (err != hipSuccess) return err;
  }
  auto launch = [&](auto kernel) {
    kernel<<<grid, block, lds, s>>>((const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N, a.K, p.tiles_m, p.tiles_n,
                                    p.split_k, p.kt_per_split, partial, a.norm_eps, ssq_part);
  };
  const bool once = weights_once(a, p.tiles_m);
  if constexpr (TM <= 5) {
    if (once) launch(a.fused_norm ? &gemm_ring_kernel<TM, TN, R, OCC, NW, 1, PIPE_NORM, 1>
                                  : &gemm_ring_kernel<TM, TN, R, OCC, NW, 0, PIPE, 1>);
  }
  if (TM > 5 || !once)
    launch(a.fused_norm ? &gemm_ring_kernel<TM, TN, R, OCC, NW, 1, PIPE_NORM, 0>
                        : &gemm_ring_kernel<TM, TN, R, OCC, NW, 0, PIPE, 0>);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || p.split_k == 1) return err;
  return launch_split_finish(partial, a.fused_norm ? ssq_part : nullptr, e, p.split_k, a, s);
}

}  // namespace
}  // namespace sf
