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
#include "sf_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

namespace sf {
namespace {

constexpr int BK = 64;
constexpr int LDK = 72;  // padded LDS row length in bf16 elements (144 B)
constexpr int XCDS = 8;

// Where a workgroup's finished accumulators go.
struct Epilogue {
  const bf16_t *bias;    // [N] or null
  const void *residual;  // [M][N] bf16, or float when res_f32; may alias y
  void *y;               // [M][N] bf16, or float when out_f32; null: not stored (arg-max partials only)
  bf16_t *y2;            // optional bf16 copy of y
  bf16_t *hooks;         // optional: bf16 copies of block row (r / hook_q, r % hook_q) into the groups of hook_mask
  float *am_val;         // optional [M][am_stride]: per row and column tile the largest value ...
  int32_t *am_idx;       // ... and its column
  int hook_mask, hook_q, hook_qmax, am_stride;
  int out_f32, res_f32, glu;
  int vec;               // every pointer above is 16-byte aligned
};

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

// 8 consecutive elements as floats; vec: every pointer of the launch is 16-byte aligned
__device__ __forceinline__ void load8(const bf16_t *p, float (&v)[8], int vec) {
  if (vec) {
    const u32x4 w = *reinterpret_cast<const u32x4 *>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[2 * i] = __uint_as_float(w[i] << 16); v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
  } else {
    for (int i = 0; i < 8; ++i) v[i] = bf2f(p[i]);
  }
}
__device__ __forceinline__ void load8(const float *p, float (&v)[8], int vec) {
  if (vec) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x4 q = *reinterpret_cast<const f32x4 *>(p + j * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j * 4 + i] = q[i];
    }
  } else {
    for (int i = 0; i < 8; ++i) v[i] = p[i];
  }
}
__device__ __forceinline__ void store8(bf16_t *p, const float (&v)[8], int vec) {
  if (vec) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack2bf(v[2 * i], v[2 * i + 1]);
    *reinterpret_cast<u32x4 *>(p) = w;
  } else {
    for (int i = 0; i < 8; ++i) p[i] = f2bf(v[i]);
  }
}
__device__ __forceinline__ void store8(float *p, const float (&v)[8], int vec) {
  if (vec) {
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<f32x4 *>(p + j * 4) = f32x4{v[j * 4], v[j * 4 + 1], v[j * 4 + 2], v[j * 4 + 3]};
  } else {
    for (int i = 0; i < 8; ++i) p[i] = v[i];
  }
}

// 8 finished columns of an output row: y, its bf16 copy, the hooked copies
__device__ __forceinline__ void store_row8(const Epilogue &e, int row, int col, int N, const float (&r)[8]) {
  const size_t o = (size_t)row * N + col;
  if (e.out_f32) store8(reinterpret_cast<float *>(e.y) + o, r, e.vec);
  else store8(reinterpret_cast<bf16_t *>(e.y) + o, r, e.vec);
  if (e.y2) store8(e.y2 + o, r, e.vec);
  if (e.hooks) {
    const size_t hrow = ((size_t)(row / e.hook_q) * e.hook_qmax + row % e.hook_q) * 4;
#pragma unroll
    for (int g = 1; g < 4; ++g)
      if (e.hook_mask >> g & 1) store8(e.hooks + (hrow + g) * N + col, r, e.vec);
  }
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
// scratch: LDS the main loop no longer needs, at least NW * BM * 8 (arg-max partials) and NW * 128 * TURN_STRIDE bytes.
template <int TM, int TN, int NW = 4>
__device__ __forceinline__ void gemm_finish(f32x16 (&acc)[TM][TN], const Epilogue &e, int M, int N, int split_k,
                                            float *__restrict__ partial, int tn, int ks, int m0, int nb0,
                                            void *scratch, float *sS = nullptr, float *__restrict__ ssq_part = nullptr,
                                            int K = 1, float eps = 0.f) {
  constexpr int BM = TM * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ln = lane & 31, lh = lane >> 5;

  // A lane holds one column of 16 rows of every 32x32 tile; stored from there, an element is a 2- or 4-byte store
  // of its own, and those stores cost more than the K loop of a short layer (160 x 2048 x 512 on 160-row tiles:
  // 20.1 us, 11.1 us this way).  So each wave turns its tiles through a private piece of LDS, one after the other,
  // and lane l then holds 16 consecutive columns of row l / 2: residual, output and copies move in 16-byte units.
  float *turn = reinterpret_cast<float *>(scratch) + wave * (32 * TURN_STRIDE);
  const int t_row = lane >> 1, t_col = (lane & 1) * 16;
  auto transpose = [&](const f32x16 &c, int col0, float (&v)[16], int step) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);  // tile by tile: overlapping them would cost registers the tall tiles lack
#pragma unroll
    for (int i = 0; i < 16; ++i) turn[c_row(i, lh) * TURN_STRIDE + ln] = c[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 q = *reinterpret_cast<const f32x4 *>(turn + t_row * TURN_STRIDE + col0 + (j >> 1) * step + (j & 1) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[j * 4 + i] = q[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  if (split_k > 1) {
    if (sS && tn == 0 && tid < BM && m0 + tid < M) ssq_part[(size_t)ks * M + m0 + tid] = sS[tid];
    __syncthreads();  // the other waves are done with the LDS this one is about to write
    static_for<TM * TN>([&](auto i_c) {
      constexpr int a = decltype(i_c)::value / TN, b = decltype(i_c)::value % TN;
      float v[16];
      transpose(acc[a][b], t_col, v, 8);
      const int row = m0 + a * 32 + t_row, col = (nb0 + b) * 32 + t_col;
      float *o = partial + ((size_t)ks * M + row) * N + col;
      if (row < M && col < N) store8(o, reinterpret_cast<const float(&)[8]>(v[0]), 1);
      if (row < M && col + 8 < N) store8(o + 8, reinterpret_cast<const float(&)[8]>(v[8]), 1);
    });
    return;
  }

  if (sS && tid < BM) sS[tid] = 1.0f / sqrtf(sS[tid] / (float)K + eps);  // one row factor per row, once

  if (e.am_val) {
    // Arg-max partials of this workgroup's column tile: per row the largest accumulator and the lowest
    // column that holds it.  Columns past N and NaN never take part.
    float *s_val = reinterpret_cast<float *>(scratch);       // [NW][BM]
    int32_t *s_idx = reinterpret_cast<int32_t *>(s_val + NW * BM);
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
          s_val[wave * BM + a * 32 + c_row(v, lh)] = best_v;
          s_idx[wave * BM + a * 32 + c_row(v, lh)] = best_i;
        }
      }
    __syncthreads();
    if (tid < BM && m0 + tid < M) {
      float bv = s_val[tid];
      int32_t bi = s_idx[tid];
#pragma unroll
      for (int w = 1; w < NW; ++w) {  // waves hold ascending column ranges
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
  auto scale_row = [&](int a, float (&v)[16]) __attribute__((always_inline)) {
    if (!sS) return;
    const float f = sS[a * 32 + t_row];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] *= f;
  };
  if (e.glu) {
    // SwiGLU.  The weight was packed with gate and up rows interleaved 16 by 16: columns 0-15 of a tile are gate
    // features f..f+15, columns 16-31 the matching up features.  Lane l takes 8 features of both.
    const int F = N >> 1;
    static_for<TM * TN>([&](auto i_c) {
      constexpr int a = decltype(i_c)::value / TN, b = decltype(i_c)::value % TN;
      const int col = (nb0 + b) * 16 + (lane & 1) * 8, row = m0 + a * 32 + t_row;
      float v[16];
      transpose(acc[a][b], (lane & 1) * 8, v, 16);
      scale_row(a, v);
      float r[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = v[i] / (1.0f + __expf(-v[i])) * v[8 + i];
      if (row < M && col < F) store8(reinterpret_cast<bf16_t *>(e.y) + (size_t)row * F + col, r, e.vec);
    });
    return;
  }

  // The residual values of a group of tiles are requested before the group's first store (y may be the residual
  // buffer itself): one exposed round trip per group.  A wave with up to five tiles forms one group, taller ones
  // go five, the tallest (no registers to spare) two tiles at a time.
  auto load_residual = [&](int a, int b, float (&res)[16]) __attribute__((always_inline)) {
    const int row = min(m0 + a * 32 + t_row, M - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const size_t o = (size_t)row * N + min((nb0 + b) * 32 + t_col + j * 8, N - 8);
      float(&dst)[8] = reinterpret_cast<float(&)[8]>(res[j * 8]);
      if (e.res_f32) load8(reinterpret_cast<const float *>(e.residual) + o, dst, e.vec);
      else load8(reinterpret_cast<const bf16_t *>(e.residual) + o, dst, e.vec);
    }
  };
  auto store_tile = [&](int a, int b, const f32x16 &c, const float (&res)[16]) __attribute__((always_inline)) {
    float v[16];
    transpose(c, t_col, v, 8);
    scale_row(a, v);
    const int row = m0 + a * 32 + t_row;
    if (row >= M) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = (nb0 + b) * 32 + t_col + j * 8;
      if (col >= N) continue;
      float r[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) r[i] = v[j * 8 + i];
      if (e.bias) {
        float bv[8];
        load8(e.bias + col, bv, e.vec);
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] += bv[i];
      }
      if (e.residual) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] += res[j * 8 + i];
      }
      store_row8(e, row, col, N, r);
    }
  };
  // constant tile indices whatever the size of the body: an unroll pragma gives up beyond a size threshold, and a
  // run-time index into the accumulators would move them out of registers
  constexpr int MOST = TM * TN > 7 ? 2 : 5;  // tiles per group
  constexpr int AG = TN >= MOST ? 1 : (TM < MOST / TN ? TM : MOST / TN), GROUPS = (TM + AG - 1) / AG;
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
template <int TM, int TN, int R, int OCC, int NW, int NORM, int PIPE = 0>
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
        wr[s][b] = Wp[((size_t)nb * k_steps + kstep) * 64 + lane];
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
            w[r][s][b] = Wp[((size_t)nb * k_steps + kstep) * 64 + lane];
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
            w[r][s][b] = Wp[((size_t)nb * k_steps + kstep) * 64 + lane];
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
    load8(p + s * step, q, 1);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] += q[i];
    if (e.glu) {
      load8(p + s * step + 16, q, 1);
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
    store8(reinterpret_cast<bf16_t *>(e.y) + (size_t)row * (N >> 1) + col, r, e.vec);
    return;
  }
  const size_t o = (size_t)row * N + col;
  if (e.bias) {
    float bv[8];
    load8(e.bias + col, bv, e.vec);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] += bv[i];
  }
  if (e.residual) {
    float res[8];
    if (e.res_f32) load8(reinterpret_cast<const float *>(e.residual) + o, res, e.vec);
    else load8(reinterpret_cast<const bf16_t *>(e.residual) + o, res, e.vec);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] += res[i];
  }
  store_row8(e, row, col, N, r);
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

struct Plan {
  int tiles_m, tiles_n, split_k, kt_per_split;
  size_t partial_bytes;
};

// split_k workgroups share a tile's K range.  The partition depends on K and split only -- never on
// the tile configuration -- because it fixes the fp32 summation order of every output element.
Plan make_plan(int M, int N, int K, int BM, int BN, int split) {
  Plan p;
  p.tiles_m = (M + BM - 1) / BM;
  p.tiles_n = (N + BN - 1) / BN;
  const int KT = (K + BK - 1) / BK;
  const int tiles = p.tiles_m * p.tiles_n;
  const int s = split < 1 ? 1 : (split > KT ? KT : split);
  p.kt_per_split = (KT + s - 1) / s;
  p.split_k = (KT + p.kt_per_split - 1) / p.kt_per_split;
  p.partial_bytes = p.split_k > 1 ? (size_t)tiles * p.split_k * BM * BN * sizeof(float) : 0;
  return p;
}

// workspace: [row sums of squares of the fused norm][partial tiles]
bool plan_fits(const Plan &p, int BM, const void *ws, size_t ws_bytes) {
  if (p.split_k == 1) return true;
  const size_t ssq_bytes = (size_t)p.tiles_m * p.split_k * BM * sizeof(float);
  return ws && ws_bytes >= GEMM_SSQ_BYTES + p.partial_bytes && ssq_bytes <= GEMM_SSQ_BYTES;
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
  hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_ring_kernel<TM, TN, R, OCC, NW, 1, PIPE_NORM>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, cap);
  if (err == hipSuccess)
    err = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_ring_kernel<TM, TN, R, OCC, NW, 0, PIPE>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, cap);
  if (err == hipSuccess) raised[dev] = true;
  return err;
}

// mode 0: launch; mode 1: only report whether (split) fits the workspace
// PIPE: issue order of the plain kernel, PIPE_NORM: of the one with the fused norm
template <int TM, int TN, int R, int OCC, int NW, int PIPE = 0, int PIPE_NORM = PIPE>
hipError_t run_ring(const GemmArgs &a, hipStream_t s, int split, int mode) {
  constexpr int BM = TM * 32, BN = NW * TN * 32;
  const Plan p = make_plan(a.M, a.N, a.K, BM, BN, split);
  if (!plan_fits(p, BM, a.ws, a.ws_bytes)) return hipErrorInvalidValue;
  if (mode == 1) return hipSuccess;
  const int groups = (p.tiles_n * p.split_k + XCDS - 1) / XCDS;  // (column tile, K split) units per XCD
  const size_t lds = lds_bytes<TM, NW>(a.fused_norm != 0);
  float *ssq_part = p.split_k > 1 ? (float *)a.ws : nullptr;
  float *partial = p.split_k > 1 ? (float *)((char *)a.ws + GEMM_SSQ_BYTES) : nullptr;
  const dim3 grid(groups * XCDS * p.tiles_m), block(64 * NW);
  if (a.am_val && (p.split_k != 1 || a.am_stride < p.tiles_n || a.fused_norm)) return hipErrorInvalidValue;
  if (a.am_val && a.am_parts_out) *a.am_parts_out = p.tiles_n;
  static_assert((size_t)2 * BM * LDK * sizeof(bf16_t) >= (size_t)NW * BM * 8, "arg-max partials fit the activation tile");
  const Epilogue e{(const bf16_t *)a.bias, a.residual, a.y, (bf16_t *)a.y2, (bf16_t *)a.hooks, a.am_val, a.am_idx,
                   a.hook_mask, a.hook_q, a.hook_qmax, a.am_stride, a.out_f32, a.res_f32, a.glu,
                   (((uintptr_t)a.bias | (uintptr_t)a.residual | (uintptr_t)a.y | (uintptr_t)a.y2 | (uintptr_t)a.hooks) & 15) == 0};
  if (lds > 64 * 1024) {
    const hipError_t err = ensure_lds<TM, TN, R, OCC, NW, PIPE, PIPE_NORM>();
    if (err != hipSuccess) return err;
  }
  if (a.fused_norm) {
    gemm_ring_kernel<TM, TN, R, OCC, NW, 1, PIPE_NORM><<<grid, block, lds, s>>>(
        (const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N, a.K, p.tiles_m, p.tiles_n, p.split_k, p.kt_per_split,
        partial, a.norm_eps, ssq_part);
  } else {
    gemm_ring_kernel<TM, TN, R, OCC, NW, 0, PIPE><<<grid, block, lds, s>>>(
        (const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N, a.K, p.tiles_m, p.tiles_n, p.split_k, p.kt_per_split,
        partial, 0.f, nullptr);
  }
  if (p.split_k > 1) {
    const int units = a.M * ((a.glu ? a.N / 2 : a.N) / 8);
    split_finish_kernel<<<(units + 255) / 256, 256, 0, s>>>(partial, a.fused_norm ? ssq_part : nullptr, e, p.split_k,
                                                            a.M, a.N, a.K, a.norm_eps);
  }
  return hipGetLastError();
}

// Tile configurations: rows per workgroup TM*32, columns NW*32 (one 32-column block per wave).
//   id  TM  ring  wg/CU  waves      (11-14: tall tiles for wide layers, see pick_large)
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
hipError_t dispatch(int tile, const GemmArgs &a, hipStream_t s, int split, int mode) {
  switch (tile) {
    case 1: return run_ring<1, 1, 4, 4, 4>(a, s, split, mode);
    case 2: return run_ring<2, 1, 4, 3, 4>(a, s, split, mode);
    case 3: return run_ring<3, 1, 4, 2, 4, 1>(a, s, split, mode);
    case 4: return run_ring<4, 1, 2, 2, 4, 1>(a, s, split, mode);
    case 5: return run_ring<5, 1, 2, 2, 4, 1>(a, s, split, mode);
    case 6: return run_ring<2, 1, 2, 1, 8, 1>(a, s, split, mode);
    case 7: return run_ring<3, 1, 4, 1, 8, 1>(a, s, split, mode);
    case 8: return run_ring<4, 1, 2, 1, 8, 1>(a, s, split, mode);
    case 9: return run_ring<5, 1, 3, 1, 8>(a, s, split, mode);
    case 10: return run_ring<5, 1, 2, 1, 8, 1>(a, s, split, mode);
    case 11: return run_ring<10, 1, 2, 1, 8, 2, 0>(a, s, split, mode);
    case 12: return run_ring<8, 1, 2, 1, 8, 2, 0>(a, s, split, mode);
    case 13: return run_ring<7, 1, 2, 1, 8>(a, s, split, mode);
    case 14: return run_ring<6, 1, 3, 1, 8>(a, s, split, mode);
    default: return hipErrorInvalidValue;
  }
}
constexpr int N_TILES = 14, N_MODEL_TILES = 10;
constexpr int TILE_TM[N_TILES + 1] = {0, 1, 2, 3, 4, 5, 2, 3, 4, 5, 5, 10, 8, 7, 6};

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
// the same sweeps.  Over the 32 shapes of that repeat the choice (this model, then the tall-tile rule) is
// the fastest measured configuration of every shape.
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
    for (int tile = N_MODEL_TILES + 1; tile <= N_TILES; ++tile) {  // 320, 256, 224, 192 rows
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

}  // namespace

// Called when weights are bound (outside any stream capture): the attribute calls of the tall tiles are
// then out of the way of the first launch.
hipError_t gemm_prepare_device() {
  hipError_t err = ensure_lds<10, 1, 2, 1, 8, 2, 0>();
  if (err == hipSuccess) err = ensure_lds<8, 1, 2, 1, 8, 2, 0>();
  if (err == hipSuccess) err = ensure_lds<7, 1, 2, 1, 8>();
  if (err == hipSuccess) err = ensure_lds<6, 1, 3, 1, 8>();
  return err;
}

int gemm_num_tiles() { return N_TILES; }
int gemm_tile_rows(int tile) { return tile >= 1 && tile <= N_TILES ? TILE_TM[tile] * 32 : 0; }

GemmConfig gemm_heuristic(int M, int plan_M, int N, int K, size_t ws_bytes) {
  // The split factor is decided for plan_M rows and then kept for any M, so a row's result does
  // not depend on how many other rows share the launch; the tile follows the actual M.
  const int split = pick(std::max(plan_M, M), N, K, ws_bytes, 0).split;
  return pick(M, N, K, ws_bytes, split);
}

bool gemm_config_fits(const GemmConfig &c, const GemmArgs &a) {
  return dispatch(c.tile, a, nullptr, c.split, 1) == hipSuccess;
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

hipError_t launch_gemm_bf16(const GemmArgs &a, hipStream_t s) {
  GemmConfig c = {a.tile, a.am_val ? 1 : a.split};  // arg-max partials: one workgroup owns a tile's whole K range
  if (c.tile <= 0 || c.split <= 0) {
    const GemmConfig h = gemm_heuristic(a.M, a.plan_M > 0 ? a.plan_M : a.M, a.N, a.K, a.ws ? a.ws_bytes : 0);
    if (c.split <= 0) c.split = h.split;
    if (c.tile <= 0) c.tile = c.split == h.split ? h.tile : pick(a.M, a.N, a.K, a.ws ? a.ws_bytes : 0, c.split).tile;
  }
  return dispatch(c.tile, a, s, c.split, 0);
}

}  // namespace sf
