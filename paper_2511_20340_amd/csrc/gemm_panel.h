// bf16 linear layers of many rows, wide: four waves, one per SIMD, each with a tile of up to 160 x 128.
//
// What bounds these layers is the card's power: under matrix load the clock falls until the power fits (a loop of nothing
// but 32x32x16 products on random operands runs at 1.74 GHz and 1.65 PFLOP/s, one of 16x16x32 products at 1.72 PFLOP/s;
// on zeros both run at 2.4 GHz), so what counts is what a product costs besides itself.  Against the block kernel, whose
// eight waves hold 160 x 64 each:
//   * a fragment read from LDS is used 8 or 10 times instead of 2 or 5: 320 x 256 rows and columns take 74 KiB of LDS reads
//     per 32 positions of K instead of 115;
//   * the 16x16x32 form moves its accumulators half as often per product (and adds over K as the 32-row form does: the bits
//     are those of the other kernels);
//   * the weights are the products' first operand: a lane then holds four consecutive columns of a row, and the epilogue
//     turns its tiles through LDS in 16-byte units, several in flight.
// With one wave on a SIMD nothing hides what the wave itself does between products, so the order is written out: after
// every product at most one LDS read or one load.  On the two largest tiles loads go out four products apart: at two apart
// they queue up in front of the L1 and 2048 x 8192 x 8192 takes 199 us instead of 187; on the others two apart (640 x 27648 x
// 5120 on 192 x 256 214 -> 198 us).
//
// The smaller tiles serve layers whose workgroups just fill the chip once: there the time of a slice is the wait for its
// loads, so three or four slices are kept in LDS (640 x 5120 x 5120: 128 x 128 with two 65 us, with four 45.6; the block
// kernel 53), or two workgroups share a compute unit.
#pragma once
#include "gemm_block.h"

namespace sf {
namespace {

// Tiles that stay in accumulation registers.  They hold 64, but with all of them taken the compiler moves one about in the
// loop, and it does not know when a product written out below is done.
constexpr int IN_ACC = 56;

// WM x WN waves, each with TM x TN tiles of 16 x 16; STAGES slices of 64 positions of K in LDS.
template <int WM, int WN, int TM, int TN, int STAGES>
struct PanelShape {
  static constexpr int NW = WM * WN, BM = WM * TM * 16, BN = WN * TN * 16;
  static constexpr int A_UNITS = BM / 8, UNITS = (BM + BN) / 8, PER = UNITS / NW;  // 1 KiB each; PER: loads per wave
  static constexpr int A_SLICE = A_UNITS * UNIT, SLICE = UNITS * UNIT;
  // after the loop the same LDS holds the row factors, the arg-max partials of the WN columns of waves, and per wave pieces
  // of 16 rows
  static constexpr int ROW = TN * 16 + 4, PIECE = 16 * ROW * 4, PIECES = 2;
  static constexpr size_t rows = (size_t)BM * (1 + 2 * WN) * 4;
  static constexpr size_t after = rows + (size_t)NW * PIECES * PIECE, loop = STAGES * (size_t)SLICE;
  static constexpr size_t lds = loop > after ? loop : after;
  static constexpr bool PAIR = lds <= 80 * 1024;  // two workgroups on a compute unit
  static constexpr bool HEAD = TN >= 8;           // takes LM heads: the narrow tiles are built without the arg-max
  static_assert(lds <= 160 * 1024 && TN % 4 == 0 && WN <= 4, "LDS of a compute unit; whole 32-column blocks per wave");
  static_assert(UNITS % NW == 0, "loads in flight are counted: every wave has as many");
  static_assert(TM * TN <= 80, "IN_ACC tiles in accumulation registers, the rest in vector registers");
};

#ifdef __HIP_DEVICE_COMPILE__
// c += w . x.  Written out because the compiler, given all accumulation registers to fill, moves tiles about in the loop.
// It knows what the statement reads and writes, but not how long a product takes: the loop is led in and followed by
// enough idle states, tied to the tiles so that no copy of one slips past them.  What the compiler made of it is looked at
// by a test of the built library.
template <bool ACC>
__device__ __forceinline__ void product(f32x4 &c, const bf16x8 &w, const bf16x8 &x) {
  if constexpr (ACC) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(w), "v"(x));
}
// A finished tile where it is used: left alone, the compiler fetches all tiles from the accumulation registers at once.
template <bool ACC>
__device__ __forceinline__ f32x4 finished(f32x4 &c) {
  if constexpr (ACC) asm volatile("" : "+a"(c));
  return c;
}
#endif

// store_row for whole units of W columns at any address, without a branch on the alignment (vector stores need none; a branch per
// unit holds up the stores behind it: float outputs with a residual 7 % slower)
template <int W>
__device__ __forceinline__ void store_at(bf16_t *p, const float (&v)[W]) {
  typedef uint32_t words __attribute__((ext_vector_type(W / 2)));
  typedef words words_at __attribute__((aligned(2)));
  words w;
#pragma unroll
  for (int i = 0; i < W / 2; ++i) w[i] = pack2bf(v[2 * i], v[2 * i + 1]);
  *reinterpret_cast<words_at *>(p) = w;
}
template <int W>
__device__ __forceinline__ void store_at(float *p, const float (&v)[W]) {
  typedef f32x4 f32x4_at __attribute__((aligned(4)));
#pragma unroll
  for (int j = 0; j < W; j += 4) *reinterpret_cast<f32x4_at *>(p + j) = f32x4{v[j], v[j + 1], v[j + 2], v[j + 3]};
}
template <int W>
__device__ __forceinline__ void store_row_at(const Epilogue &e, int row, int col, int N, const float (&r)[W]) {
  const size_t o = (size_t)row * N + col;
  if (e.out_f32) store_at(reinterpret_cast<float *>(e.y) + o, r);
  else store_at(reinterpret_cast<bf16_t *>(e.y) + o, r);
  if (e.y2) store_at(e.y2 + o, r);
  if (e.hooks) {
    const size_t hrow = ((size_t)(row / e.hook_q) * e.hook_qmax + row % e.hook_q) * 4;
#pragma unroll
    for (int g = 1; g < 4; ++g)
      if (e.hook_mask >> g & 1) store_at(e.hooks + (hrow + g) * N + col, r);
  }
}

template <int WM, int WN, int TM, int TN, int STAGES>
__global__ __launch_bounds__(64 * WM * WN, 1) void gemm_panel_kernel(const bf16_t *__restrict__ A, const uint4 *__restrict__ Wp,
                                                                     const Epilogue e, int M, int N, int K, int tiles_m,
                                                                     int tiles_n, int split_k, int kt_per_split,
                                                                     float *__restrict__ partial, float eps,
                                                                     const float *__restrict__ ssq) {
#ifdef __HIP_DEVICE_COMPILE__
  using S = PanelShape<WM, WN, TM, TN, STAGES>;
  constexpr int NW = S::NW, BM = S::BM, PER = S::PER;
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int id = blockIdx.x;
  const int xcd = id % XCDS, j = id / XCDS;
  // The units of an XCD and the row tiles that share a unit's weights: those side by side, or, where a compute unit holds
  // two workgroups, all units of one row tile first, so that the second half of a not quite full round spreads evenly
  // (320 x 28672 x 4096 on 160 x 128 with two: 97 us side by side, 93 this way; 1280 x 28672 x 4096 on 320 x 256 with one
  // takes 247 us this way, 230 side by side; single unsplit launches on one card, bf16 out, weights rotated).
  const int per = (tiles_n * split_k + XCDS - 1) / XCDS;
  const int tm = S::PAIR ? j / per : j % tiles_m, unit = (S::PAIR ? j % per : j / tiles_m) * XCDS + xcd;
  if (unit >= tiles_n * split_k) return;
  const int tn = unit / split_k, ks = unit % split_k;
  const int m0 = tm * BM, n0 = tn * S::BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const int n_blocks = (N + 31) >> 5, k_steps = K >> 4, KT = K / BK;
  const int kt0 = ks * kt_per_split, kt1 = min(KT, kt0 + kt_per_split);

  // This wave's loads of a slice: eight rows of activations (16-byte chunk c of row r goes to place c ^ (r & 7) of its LDS
  // row) or one packed unit of weights each.
  const buffer_t buf_a = make_buffer(A, (size_t)M * K * 2), buf_w = make_buffer(Wp, (size_t)n_blocks * k_steps * UNIT);
  uint32_t src[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int u = wave + i * NW, v = u - S::A_UNITS;
    if (v < 0) {
      const int row = u * 8 + (lane >> 3);
      src[i] = (uint32_t)min(m0 + row, M - 1) * (uint32_t)K * 2 + (((lane & 7) ^ (row & 7)) << 4);
    } else {
      src[i] = ((uint32_t)min((n0 >> 5) + (v >> 2), n_blocks - 1) * k_steps + (v & 3)) * UNIT + lane * 16;
    }
  }
  // slices past the end load the last one again: in bounds and never used
  uint32_t a_pos = kt0 * BK * 2, w_pos = kt0 * 4 * UNIT, fill = 0;
  const uint32_t a_last = (kt1 - 1) * BK * 2, w_last = (kt1 - 1) * 4 * UNIT;
  auto load = [&](auto i_c) __attribute__((always_inline)) {
    constexpr int i = decltype(i_c)::value;
    const int u = wave + i * NW;
    auto *to = (__attribute__((address_space(3))) void *)(smem + fill + u * UNIT);
    if constexpr ((i + 1) * NW <= S::A_UNITS) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(buf_a, to, 16, src[i], a_pos, 0, 0);
    } else if constexpr (i * NW >= S::A_UNITS) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(buf_w, to, 16, src[i], w_pos, 0, 0);
    } else {
      if (u < S::A_UNITS) __builtin_amdgcn_raw_ptr_buffer_load_lds(buf_a, to, 16, src[i], a_pos, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(buf_w, to, 16, src[i], w_pos, 0, 0);
    }
    if constexpr (i == PER - 1) {
      a_pos = min(a_pos + BK * 2, a_last);
      w_pos = min(w_pos + 4 * UNIT, w_last);
      fill = fill == (STAGES - 1) * S::SLICE ? 0 : fill + S::SLICE;
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragments of k-step s (32 positions) of the slice at `cur`: lane (l16, lq) holds positions 8 lq .. 8 lq + 7 of a row
  // or column
  bf16x8 fa[2][TM], fb[2][TN];
  const int a_row = (wm * TM * 16 + l16) * (BK * 2);
  const int a_lane[2] = {a_row + ((lq ^ (l16 & 7)) << 4), a_row + (((4 + lq) ^ (l16 & 7)) << 4)};
  const int w_lane = S::A_SLICE + wn * (TN / 2) * 4 * UNIT + (lane >> 5) * UNIT + (lq & 1) * 512 + l16 * 16;
  uint32_t cur = 0;
  auto read_a = [&](int s, int a) __attribute__((always_inline)) {
    fa[s][a] = *reinterpret_cast<const bf16x8 *>(smem + cur + a_lane[s] + a * 16 * BK * 2);
  };
  auto read_w = [&](int s, int b) __attribute__((always_inline)) {
    fb[s][b] = *reinterpret_cast<const bf16x8 *>(smem + cur + w_lane + s * 2 * UNIT + (b >> 1) * 4 * UNIT + (b & 1) * 256);
  };
  // Row a of a k-step is TN products with activation fragment a.  That fragment is read AHEAD rows before; the weights of
  // the next k-step in the rows from TURN on.  In the second k-step of a slice those reads are of the next slice: before
  // row TURN the waves meet, the next slice has landed, and as nobody reads this one any more the loads of the slice that
  // takes its place begin, LOAD_GAP products apart.
  constexpr int AHEAD = TN >= 8 ? (TM >= 6 ? 3 : 2) : 3, TURN = TM - AHEAD, LOAD_GAP = TM * TN >= 64 ? 4 : 2;
  constexpr int NEW = AHEAD + TN, SPACE = AHEAD * TN;  // reads in the rows from TURN on, and their products
  static_assert(TURN >= 1 && SPACE >= NEW, "reads fit between the products");
  constexpr int TAIL = SPACE / LOAD_GAP < PER ? SPACE / LOAD_GAP : PER;  // loads in the second k-step
  constexpr int GAP0 = (PER - TAIL) * LOAD_GAP <= TM * TN ? LOAD_GAP : TM * TN / (PER - TAIL);  // gap in the first
  auto k_step = [&](auto s_c) __attribute__((always_inline)) {
    constexpr int s = decltype(s_c)::value;
    static_for<TM * TN>([&](auto i_c) __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value, a = i / TN, b = i % TN;
      if constexpr (s == 1 && i == TURN * TN) {
        wait_loads_and_meet<(STAGES - 2) * PER>();
        cur = cur == (STAGES - 1) * S::SLICE ? 0 : cur + S::SLICE;
      }
      product<(i < IN_ACC)>(acc[a][b], fb[s][b], fa[s][a]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (a < TURN) {
        if constexpr (b == TN / 2) read_a(s, a + AHEAD);
      } else {  // the weights first, they are all needed in the next row 0
        constexpr int p = i - TURN * TN, n = p * NEW / SPACE, last = (p - 1 + SPACE) * NEW / SPACE - NEW;
        if constexpr (p == 0 || n != last) {
          constexpr int FIRST_A = TN - 1;  // activation 0 goes before the last weights
          if constexpr (n < FIRST_A) read_w(s ^ 1, n);
          else if constexpr (n == FIRST_A) read_a(s ^ 1, 0);
          else if constexpr (n == FIRST_A + 1) read_w(s ^ 1, TN - 1);
          else read_a(s ^ 1, n - TN);
        }
      }
      if constexpr (s == 1 && a >= TURN) {
        constexpr int p = i - TURN * TN;
        if constexpr (p % LOAD_GAP == LOAD_GAP - 1 && p / LOAD_GAP < TAIL) load(std::integral_constant<int, p / LOAD_GAP>{});
      }
      if constexpr (s == 0 && PER > TAIL) {
        if constexpr (i % GAP0 == GAP0 - 1 && i / GAP0 < PER - TAIL) load(std::integral_constant<int, TAIL + i / GAP0>{});
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  static_for<STAGES - 1>([&](auto) __attribute__((always_inline)) { static_for<PER>(load); });
  wait_loads_and_meet<(STAGES - 2) * PER>();
  static_for<TAIL>(load);
#pragma unroll
  for (int b = 0; b < TN; ++b) read_w(0, b);
#pragma unroll
  for (int a = 0; a < AHEAD; ++a) read_a(0, a);
  __builtin_amdgcn_s_waitcnt(0xc07f);
  auto pin_tiles = [&]() __attribute__((always_inline)) {
    static_for<TM * TN>([&](auto i_c) __attribute__((always_inline)) {
      constexpr int i = decltype(i_c)::value;
      f32x4 &c = acc[i / TN][i % TN];
      if constexpr (i < IN_ACC) asm volatile("" : "+a"(c));
      else asm volatile("" : "+v"(c));
    });
  };
  pin_tiles();  // the accumulators are zeroed before this point, and settled behind it
  asm volatile("s_nop 7" ::);
  __builtin_amdgcn_sched_barrier(0);
  for (int i = kt0; i < kt1; ++i) {
    k_step(std::integral_constant<int, 0>{});
    k_step(std::integral_constant<int, 1>{});
  }
  // the last products are done: the idle states hold the newest tiles (products finish in order, those before them are done
  // by then), and no tile is read ahead of them
  {
    constexpr int L = TM * TN;
    f32x4 &n1 = acc[TM - 1][TN - 1], &n2 = acc[TM - 1][TN - 2], &n3 = acc[TM - 1][TN - 3], &n4 = acc[TM - 1][TN - 4];
    static_assert(L <= IN_ACC || L >= IN_ACC + 4, "the newest four tiles are in one kind of registers");
    if constexpr (L <= IN_ACC)
      asm volatile("s_nop 15\n\ts_nop 15" : "+a"(n1), "+a"(n2), "+a"(n3), "+a"(n4));
    else
      asm volatile("s_nop 15\n\ts_nop 15" : "+v"(n1), "+v"(n2), "+v"(n3), "+v"(n4));
  }
  pin_tiles();
  // nothing may land in LDS any more, the epilogue reuses it
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  float *const sS = reinterpret_cast<float *>(smem);
  if (split_k == 1) {  // one factor per row: of the fused norm, or 1
    for (int r = tid; r < BM; r += 64 * NW) sS[r] = ssq ? 1.0f / sqrtf(ssq[min(m0 + r, M - 1)] / (float)K + eps) : 1.f;
    __syncthreads();
  }

  const int col0 = n0 + wn * TN * 16;
  if (S::HEAD && e.am_val) {
    // Arg-max partials of this workgroup's columns: a lane walks its columns in ascending order (a NaN is never greater),
    // the four lanes of a row and the WN waves compare value, then column.  Columns past N never take part.
    float *s_val = sS + BM;                                      // [WN][BM]
    int32_t *s_idx = reinterpret_cast<int32_t *>(s_val + WN * BM);  // [WN][BM]
    auto better = [](float v, int32_t i, float bv, int32_t bi) __attribute__((always_inline)) {
      return i != INT32_MAX && (bi == INT32_MAX || v > bv || (v == bv && i < bi));
    };
    static_for<TM>([&](auto a_c) __attribute__((always_inline)) {
      constexpr int a = decltype(a_c)::value;
      float bv = -__builtin_huge_valf();
      int32_t bi = INT32_MAX;
      static_for<TN>([&](auto b_c) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value;
        const f32x4 v = finished<(a * TN + b < IN_ACC)>(acc[a][b]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int col = col0 + b * 16 + lq * 4 + i;
          const bool up = (col < N) & ((v[i] > bv) | ((bi == INT32_MAX) & (v[i] == bv)));  // no branches
          bv = up ? v[i] : bv;
          bi = up ? col : bi;
        }
      });
#pragma unroll
      for (int w = 16; w < 64; w <<= 1) {
        const float ov = __shfl_xor(bv, w);
        const int32_t oi = __shfl_xor(bi, w);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
      }
      if (lq == 0) {
        s_val[wn * BM + (wm * TM + a) * 16 + l16] = bv;
        s_idx[wn * BM + (wm * TM + a) * 16 + l16] = bi;
      }
    });
    __syncthreads();
    for (int r = tid; r < BM && m0 + r < M; r += 64 * NW) {
      float bv = s_val[r];
      int32_t bi = s_idx[r];
#pragma unroll
      for (int w = 1; w < WN; ++w)
        if (better(s_val[w * BM + r], s_idx[w * BM + r], bv, bi)) { bv = s_val[w * BM + r]; bi = s_idx[w * BM + r]; }
      e.am_val[(size_t)(m0 + r) * e.am_stride + tn] = bv;
      e.am_idx[(size_t)(m0 + r) * e.am_stride + tn] = bi;
    }
    if (!e.y) return;
  }

  // Outputs: 16 rows at a time each wave turns its tiles through a piece of LDS of its own (two, by turns); a lane then
  // holds W consecutive columns of a row, and a store instruction writes whole lines.
  char *const pieces = smem + S::rows + wave * (S::PIECES * S::PIECE);
  auto settle = []() __attribute__((always_inline)) {  // between the lanes of a wave, whose LDS accesses keep their order
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (e.glu && split_k == 1) {
    // SwiGLU: the weight was packed with gate and up rows interleaved 16 by 16, so tiles 2b and 2b + 1 hold a feature's
    // gate and up value in the same lane and register
    constexpr int RB = TN * 16 + 16;  // bytes of an LDS row: TN * 8 features and 16 to spread the banks
    const int F = N >> 1;
    static_for<TM>([&](auto a_c) __attribute__((always_inline)) {
      constexpr int a = decltype(a_c)::value;
      char *p = pieces + a % S::PIECES * S::PIECE;
      const float f = sS[(wm * TM + a) * 16 + l16];
      static_for<TN / 2>([&](auto b_c) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value * 2, t = a * TN + b;
        const f32x4 gate = finished<(t < IN_ACC)>(acc[a][b]), up = finished<(t + 1 < IN_ACC)>(acc[a][b + 1]);
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = gate[i] * f;
          r[i] = g / (1.0f + __expf(-g)) * (up[i] * f);
        }
        *reinterpret_cast<uint2 *>(p + l16 * RB + b * 16 + lq * 8) = make_uint2(pack2bf(r[0], r[1]), pack2bf(r[2], r[3]));
      });
      settle();
#pragma unroll
      for (int t = 0; t < (TN + 3) / 4; ++t) {
        const int u = t * 64 + lane, r = u / TN, c = (u - r * TN) * 8;
        const int row = m0 + (wm * TM + a) * 16 + r, col = (col0 >> 1) + c;
        if (r < 16 && row < M && col < F) {
          bf16_t *to = reinterpret_cast<bf16_t *>(e.y) + (size_t)row * F + col;
          const uint4 v = *reinterpret_cast<const uint4 *>(p + r * RB + c * 2);
          if (e.vec) {
            *reinterpret_cast<uint4 *>(to) = v;
          } else {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) to[i] = (bf16_t)(w[i >> 1] >> (i & 1) * 16);
          }
        }
      }
      settle();
    });
    return;
  }
  // how_c: PLAIN rows, a bias; FULL, FULL_BF: also a float or bf16 residual (requested as many pieces ahead as registers allow: y
  // may be the residual, a lane's own elements; at any address), bf16 copy, hooked copies; ANY: rows that end within the W, any
  // types, in a loop that is not unrolled and waits for every residual (1280 x 28672 x 4096, bf16 with bias and residual: 373
  // us that way, FULL_BF 250, another 3 % less with loops of its own below; without either 245).  A lane's units are in the same columns of every row, so it reads its bias
  // once, ahead (read for every unit, 1024 x 16384 x 256 with a bias took 21.8 us; 16.6 this way, 17.0
  // without one)
  enum { PLAIN, FULL, FULL_BF, ANY };
  auto bf_of = [](const auto &w, int i) __attribute__((always_inline)) {  // value i of packed bf16
    return __uint_as_float(i & 1 ? w[i >> 1] & 0xffff0000u : w[i >> 1] << 16);
  };
  auto outputs = [&](auto w_c, auto how_c, auto store) __attribute__((always_inline)) {
    constexpr int W = decltype(w_c)::value, PR = TN * 16 / W, T = (16 * PR + 63) / 64;  // units per row; units per lane
    constexpr int how = decltype(how_c)::value;
    constexpr bool ahead = how == FULL || how == FULL_BF;
    typedef uint32_t words __attribute__((ext_vector_type(W / 2)));
    typedef std::conditional_t<how == FULL_BF, words, f32x4> res_t;
    typedef std::conditional_t<how == FULL_BF, bf16_t, float> res_e;
    typedef res_t __attribute__((aligned(sizeof(res_e)))) res_at;
    auto place = [&](int a, int t, int &r, int &row, int &col) __attribute__((always_inline)) {
      const int u = t * 64 + lane;
      r = u / PR;
      row = m0 + (wm * TM + a) * 16 + r;
      col = col0 + (u - r * PR) * W;
    };
    constexpr int DEEP = 24 / T < 1 ? 1 : 24 / T, RING = TM < DEEP ? TM : DEEP;  // pieces of residual rows in flight
    res_t res[ahead ? RING : 1][ahead ? T : 1];
    static_assert(64 % PR == 0, "one bias per lane");
    words bias = {};
    if (how != ANY && e.bias) {
      typedef words __attribute__((aligned(2))) words_at;
      bias = *reinterpret_cast<const words_at *>(e.bias + min(col0 + lane % PR * W, N - W));
    }
    auto request = [&](int to, int a) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < T; ++t) {
        int r, row, col;
        place(a, t, r, row, col);
        res[to][t] = *reinterpret_cast<const res_at *>(reinterpret_cast<const res_e *>(e.residual) +
                                                      (size_t)min(row, M - 1) * N + min(col, N - W));
      }
    };
    auto piece = [&](int a, int t, const float *p, res_t &own) __attribute__((always_inline)) {
      int r, row, col;
      place(a, t, r, row, col);
      if ((16 * PR) % 64 != 0 && r >= 16) return;
      float v[W];
      load_n(p + r * S::ROW + (col - col0), v, 1);
      if (row < M && col < N) {
        if constexpr (ahead) store((wm * TM + a) * 16 + r, row, col, v, own, bias);
        else if constexpr (how == PLAIN) store((wm * TM + a) * 16 + r, row, col, v, bias);
        else store((wm * TM + a) * 16 + r, row, col, v);
      }
    };
    if (ahead && e.residual) {
#pragma unroll
      for (int a = 0; a < RING; ++a) request(a, a);
    }
    static_for<TM>([&](auto a_c) __attribute__((always_inline)) {
      constexpr int a = decltype(a_c)::value;
      float *p = reinterpret_cast<float *>(pieces + a % S::PIECES * S::PIECE);
      static_for<TN>([&](auto b_c) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value;
        *reinterpret_cast<f32x4 *>(p + l16 * S::ROW + b * 16 + lq * 4) = finished<(a * TN + b < IN_ACC)>(acc[a][b]);
      });
      settle();
      if constexpr (how == ANY) {
#pragma unroll 1
        for (int t = 0; t < T; ++t) piece(a, t, p, res[0][0]);
      } else {
#pragma unroll
        for (int t = 0; t < T; ++t) piece(a, t, p, res[ahead ? a % RING : 0][ahead ? t : 0]);
        if constexpr (ahead && a + RING < TM) {
          if (e.residual) request(a % RING, a + RING);
        }
      }
      settle();
    });
  };
  typedef std::integral_constant<int, 4> four;  // floats: eight lanes write a 128-byte line
  typedef std::integral_constant<int, 8> eight;
  typedef std::integral_constant<int, PLAIN> plain;
  typedef std::integral_constant<int, FULL> full;
  typedef std::integral_constant<int, FULL_BF> full_bf;
  typedef std::integral_constant<int, ANY> any;
  if (split_k > 1) {
    outputs(four{}, plain{}, [&](int, int row, int col, float (&v)[4], const auto &) __attribute__((always_inline)) {
      store_n(partial + ((size_t)ks * M + row) * N + col, v, 1);
    });
  } else if (N % 8 != 0 || (!e.out_f32 && (e.y2 || e.hooks || (e.residual && e.res_f32)))) {
    outputs(four{}, any{}, [&](int in_tile, int row, int col, float (&v)[4]) __attribute__((always_inline)) {
      const float f = sS[in_tile];
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] *= f;
      if (e.bias) {
        load_n(e.bias + col, x, e.vec);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += x[i];
      }
      if (e.residual) {
        if (e.res_f32) load_n(reinterpret_cast<const float *>(e.residual) + (size_t)row * N + col, x, e.vec);
        else load_n(reinterpret_cast<const bf16_t *>(e.residual) + (size_t)row * N + col, x, e.vec);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] += x[i];
      }
      store_row(e, row, col, N, v);
    });
  } else if (e.vec && !e.out_f32 && !e.residual) {
    auto rows = [&](auto with) __attribute__((always_inline)) {  // two loops: a branch per unit costs 1 to 2 % without a bias
      outputs(eight{}, plain{}, [&](int in_tile, int row, int col, float (&v)[8], const auto &bias) __attribute__((always_inline)) {
        const float f = sS[in_tile];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] *= f;
        if constexpr (decltype(with)::value) {
#pragma unroll
          for (int i = 0; i < 8; ++i) v[i] += bf_of(bias, i);
        }
        store_n(reinterpret_cast<bf16_t *>(e.y) + (size_t)row * N + col, v, 1);
      });
    };
    if (e.bias) rows(std::true_type{});
    else rows(std::false_type{});
  } else if (e.vec && !e.bias && !e.residual && !e.y2 && !e.hooks) {
    outputs(four{}, plain{}, [&](int in_tile, int row, int col, float (&v)[4], const auto &) __attribute__((always_inline)) {
      const float f = sS[in_tile];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] *= f;
      store_n(reinterpret_cast<float *>(e.y) + (size_t)row * N + col, v, 1);
    });
  } else {
    auto all = [&](int in_tile, int row, int col, auto &v, auto &res, const auto &bias) __attribute__((always_inline)) {
      constexpr int W = sizeof(v) / sizeof(float);
      const float f = sS[in_tile];
#pragma unroll
      for (int i = 0; i < W; ++i) v[i] *= f;
      if (e.bias) {
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] += bf_of(bias, i);
      }
      if (e.residual) {
#pragma unroll
        for (int i = 0; i < W; ++i) {
          if constexpr (std::is_same_v<std::remove_reference_t<decltype(res)>, f32x4>) v[i] += res[i];
          else v[i] += bf_of(res, i);
        }
      }
      store_row_at(e, row, col, N, v);
    };
    // a bf16 residual and nothing else but a bias: written out for either (with the branches of `all`, 2048 x 16384 x 256 into bf16
    // with both takes 42 us; 36 this way)
    auto sums = [&](auto w_c, auto with) __attribute__((always_inline)) {
      constexpr int W = decltype(w_c)::value;
      typedef std::conditional_t<W == 8, bf16_t, float> out_t;
      outputs(w_c, full_bf{}, [&](int in_tile, int row, int col, float (&v)[W], auto &res, const auto &bias) __attribute__((always_inline)) {
        const float f = sS[in_tile];
#pragma unroll
        for (int i = 0; i < W; ++i) {
          v[i] *= f;
          if constexpr (decltype(with)::value) v[i] += bf_of(bias, i);
          v[i] += bf_of(res, i);
        }
        store_at(reinterpret_cast<out_t *>(e.y) + (size_t)row * N + col, v);
      });
    };
    if (e.residual && !e.res_f32 && !e.y2 && !e.hooks) {
      if (e.out_f32) {
        if (e.bias) sums(four{}, std::true_type{});
        else sums(four{}, std::false_type{});
      } else {
        if (e.bias) sums(eight{}, std::true_type{});
        else sums(eight{}, std::false_type{});
      }
    } else if (!e.out_f32) {
      outputs(eight{}, full_bf{}, all);
    } else if (e.residual && !e.res_f32) {
      outputs(four{}, full_bf{}, all);
    } else {
      outputs(four{}, full{}, all);
    }
  }
#endif
}

template <int WM, int WN, int TM, int TN, int STAGES>
hipError_t ensure_panel_lds() {
  constexpr int cap = (int)PanelShape<WM, WN, TM, TN, STAGES>::lds;
  if (cap <= 64 * 1024) return hipSuccess;
  static bool raised[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (raised[dev]) return hipSuccess;
  const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_panel_kernel<WM, WN, TM, TN, STAGES>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, cap);
  if (err == hipSuccess) raised[dev] = true;
  return err;
}

template <int WM, int WN, int TM, int TN, int STAGES>
hipError_t run_panel(const GemmArgs &a, hipStream_t s, int split) {
  using S = PanelShape<WM, WN, TM, TN, STAGES>;
  const Plan p = make_plan(a.M, a.N, a.K, S::BM, S::BN, split);
  const bool two = p.split_k > 1;  // a second launch adds the partial tiles
  if (!plan_fits(p, S::BM, a.ws, a.ws_bytes) || (a.fused_norm && !two && !squares_fit(a.M, gemm_norm_bytes(a)))) return hipErrorInvalidValue;
  const int groups = (p.tiles_n * p.split_k + XCDS - 1) / XCDS;
  float *partial = two ? (float *)((char *)a.ws + GEMM_SSQ_BYTES) : nullptr;
  if (a.am_val && (!S::HEAD || p.split_k != 1 || a.am_stride < p.tiles_n || a.fused_norm)) return hipErrorInvalidValue;
  if (a.am_val && a.am_parts_out) *a.am_parts_out = p.tiles_n;
  const Epilogue e = make_epilogue(a);
  hipError_t err = ensure_panel_lds<WM, WN, TM, TN, STAGES>();
  float *ssq = a.fused_norm ? (float *)a.ws : nullptr;  // [split][M]
  if (err == hipSuccess && ssq) err = launch_row_squares(a, p.split_k, p.kt_per_split, ssq, s);
  if (err != hipSuccess) return err;
  gemm_panel_kernel<WM, WN, TM, TN, STAGES><<<groups * XCDS * p.tiles_m, 64 * S::NW, S::lds, s>>>(
      (const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N, a.K, p.tiles_m, p.tiles_n, p.split_k, p.kt_per_split, partial,
      a.norm_eps, two ? nullptr : ssq);
  err = hipGetLastError();
  if (err != hipSuccess || !two) return err;
  return launch_split_finish(partial, ssq, e, p.split_k, a, s);
}

}  // namespace
}  // namespace sf
