// bf16 linear layers of many rows: both operands through LDS, filled by direct global -> LDS loads.
//
// In the ring kernel (gemm_ring.h) every wave streams its own weights to registers and reads the whole activation tile
// from LDS for one column block: per product of two 32x32x16 fragments it moves a KiB through LDS, the activations pass
// through registers on their way there, and its tallest tiles have no registers left to hide either.  Here the waves of a
// workgroup stand in a WM x WN grid, each with TM x TN tiles, so a fragment read from LDS is used TN or TM times; neither
// operand passes through registers on its way to LDS, so what is in flight is bounded by the 160 KiB of LDS alone; the
// packed weight units are LDS fragments as they are.  Activations arrive in rows of whole 128-byte lines (64-byte pieces
// of half as long slices cost 4 to 10 % more).
// What bounds it: operand latency.  512 x 2048 x 2048 9.7 us (ring kernel 16.7), 320 x 5120 x 13824 67 (88).  The largest
// tiles are the panel kernel's (gemm_panel.h): 1280 x 28672 x 4096 with the norm 272 us on eight waves here, 238 there.
//
// Same products in the same order, same K partition, same row sums as the ring kernel: the same bits.
//
// Small layers with their K split: instead of leaving partial tiles to a second launch (5 us of a 15 us layer), KG groups
// of waves in one workgroup take a part of K each and the first adds the others' sums from LDS, in split order.
// 160 x 3072 x 2048 with the norm in 2 parts: 17.6 us (ring kernel + second launch) -> 9.4; 160 x 2048 x 2048 14.7 -> 7.7;
// 61 x 6144 x 4096 20.7 -> 18.6.
#pragma once
#include "gemm_ring.h"

namespace sf {
namespace {

constexpr int BS = 32;          // K positions of a weight slice (the activations move BK at a time: whole 128-byte lines)
constexpr int UNIT = 1024;      // bytes one wave-wide 16-byte load moves

#ifdef __HIP_DEVICE_COMPILE__  // the host pass knows neither the descriptor type nor the loads
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t make_buffer(const void *p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (uint32_t)bytes, 0x00020000);
}

template <int N>
__device__ __forceinline__ void wait_loads_and_meet() {  // all but the N newest loads have landed, own LDS reads are done
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
#endif

// WM x WN waves, TM x TN 32x32 tiles each; STAGES slices of BK positions in LDS.  KG groups of such waves share the K of a
// split layer among themselves, each with its own slices.
template <int WM, int WN, int TM, int TN, int STAGES, int KG = 1>
struct BlockShape {
  static constexpr int NW = WM * WN, BM = WM * TM * 32, BN = WN * TN * 32;
  static constexpr int A_SLICE = BM * BK * 2, W_SLICE = BN * BS * 2, W0 = STAGES * A_SLICE;  // bytes; W0: the weights' place
  static constexpr int A_PER = (A_SLICE / UNIT + NW - 1) / NW, W_PER = (W_SLICE / UNIT + NW - 1) / NW;  // loads per wave
  // after the loop the same LDS holds the epilogue's pieces, then the fused norm's row factors and sums by chunk
  static constexpr size_t turn = (size_t)NW * 32 * TURN_STRIDE * 4;
  static constexpr size_t sums = (size_t)(KG - 1) * BM * BN * 4 > turn ? (size_t)(KG - 1) * BM * BN * 4 : turn;  // or the groups' sums
  static constexpr size_t after = sums + (size_t)BM * (1 + 8 * KG) * 4;
  static constexpr size_t group = (size_t)W0 + 2 * STAGES * W_SLICE, loop = KG * group, lds = loop > after ? loop : after;
  static_assert(lds <= 160 * 1024 && turn >= (size_t)WN * BM * 8, "LDS of a compute unit; arg-max partials");
};

template <int WM, int WN, int TM, int TN, int STAGES, int KG, int NORM>
__global__ __launch_bounds__(64 * WM * WN * KG) void gemm_block_kernel(const bf16_t *__restrict__ A, const uint4 *__restrict__ Wp,
                                                                    const Epilogue e, int M, int N, int K, int tiles_m,
                                                                    int tiles_n, int split_k, int kt_per_split,
                                                                    float *__restrict__ partial, float eps,
                                                                    float *__restrict__ ssq_part) {
#ifdef __HIP_DEVICE_COMPILE__
  using S = BlockShape<WM, WN, TM, TN, STAGES, KG>;
  constexpr int NW = S::NW, BM = S::BM, A_PER = S::A_PER, W_PER = S::W_PER;
  extern __shared__ __attribute__((aligned(1024))) char smem_all[];

  const int id = blockIdx.x;
  const int xcd = id % XCDS, j = id / XCDS;
  const int tm = j % tiles_m, unit = (j / tiles_m) * XCDS + xcd;
  if (unit >= (KG == 1 ? tiles_n * split_k : tiles_n)) return;
  const int m0 = tm * BM;
  const int tid = threadIdx.x, lane = tid & 63, any_wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = KG == 1 ? 0 : any_wave / NW, wave = KG == 1 ? any_wave : any_wave % NW;
  const int tn = KG == 1 ? unit / split_k : unit, ks = KG == 1 ? unit % split_k : kg;
  char *const smem = smem_all + kg * S::group;
  const int ln = lane & 31, lh = lane >> 5;
  const int wm = wave / WN, wn = wave % WN;
  const int n_blocks = (N + 31) >> 5, k_steps = K >> 4, KT = K / BK;
  const int kt0 = ks * kt_per_split, kt1 = min(KT, kt0 + kt_per_split);
  const int n = kt1 - kt0;  // activation slices; twice as many weight slices
  const int rounds = KG == 1 ? n : kt_per_split;  // the last group may have fewer slices than meetings

  // this wave's loads of a slice: eight rows of activations, or one packed unit of weights each.  16-byte chunk c of row
  // r of the activations goes to place c ^ (r & 7) of its LDS row, so that the 32 rows a fragment read touches spread
  // over the banks.
  const buffer_t buf_a = make_buffer(A, (size_t)M * K * 2), buf_w = make_buffer(Wp, (size_t)n_blocks * k_steps * UNIT);
  uint32_t a_src[A_PER], w_src[W_PER], a_dst[A_PER], w_dst[W_PER];
#pragma unroll
  for (int i = 0; i < A_PER; ++i) {
    const int u = min(wave + i * NW, S::A_SLICE / UNIT - 1), row = u * 8 + (lane >> 3);
    a_dst[i] = u * UNIT;
    a_src[i] = (uint32_t)min(m0 + row, M - 1) * (uint32_t)K * 2 + (((lane & 7) ^ (row & 7)) << 4);
  }
#pragma unroll
  for (int i = 0; i < W_PER; ++i) {
    const int u = min(wave + i * NW, S::W_SLICE / UNIT - 1), nb = min(tn * WN * TN + (u >> 1), n_blocks - 1);
    w_dst[i] = S::W0 + u * UNIT;
    w_src[i] = ((uint32_t)nb * k_steps + (u & 1)) * UNIT + lane * 16;
  }
  // slices past the end load the last one again: in bounds, never used, and the counts of loads in flight stay the same
  uint32_t a_pos = kt0 * BK * 2, w_pos = kt0 * 4 * UNIT, a_fill = 0, w_fill = 0;
  const uint32_t a_last = (kt1 - 1) * BK * 2, w_last = (kt1 * 4 - 2) * UNIT;
  auto load_a = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < A_PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(buf_a, (__attribute__((address_space(3))) void *)(smem + a_fill + a_dst[i]), 16,
                                               a_src[i], a_pos, 0, 0);
    a_pos = min(a_pos + BK * 2, a_last);
    a_fill = a_fill == (STAGES - 1) * S::A_SLICE ? 0 : a_fill + S::A_SLICE;
  };
  auto load_w = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < W_PER; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(buf_w, (__attribute__((address_space(3))) void *)(smem + w_fill + w_dst[i]), 16,
                                               w_src[i], w_pos, 0, 0);
    w_pos = min(w_pos + 2 * UNIT, w_last);
    w_fill = w_fill == (2 * STAGES - 1) * S::W_SLICE ? 0 : w_fill + S::W_SLICE;
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  bf16x8 fa[2][TM], fb[2][TN];
  const int a_lane = (wm * TM * 32 + ln) * (BK * 2), w_lane = S::W0 + wn * TN * 2 * UNIT + lane * 16;
  uint32_t a_cur = 0, w_cur = 0;
  auto fragments = [&](int to, int s) __attribute__((always_inline)) {  // k-step s of the current activation slice
    const char *pa = smem + a_cur + (a_lane + (((2 * s + lh) ^ (ln & 7)) << 4)), *pw = smem + w_cur + w_lane + (s & 1) * UNIT;
#pragma unroll
    for (int b = 0; b < TN; ++b) fb[to][b] = *reinterpret_cast<const bf16x8 *>(pw + b * 2 * UNIT);
#pragma unroll
    for (int a = 0; a < TM; ++a) fa[to][a] = *reinterpret_cast<const bf16x8 *>(pa + a * 32 * BK * 2);
  };
  // Fused norm: of the WN waves that multiply the same rows, wave wn squares the fragments of k-step wn (and wn + WN):
  // each lane sums one 16-byte chunk of a row over the slices, in the order of the ring kernel, so both leave the same bits.
  constexpr int SQ = WN >= 4 ? 1 : 4 / WN;  // k-steps per wave
  // waves w and w + 4 share a SIMD: they take different k-steps, so one multiplies while the other squares
  const int sq_wn = WN == 4 ? (wn + 2 * wm) % 4 : wn;
  float ssq[SQ][TM];
#pragma unroll
  for (int i = 0; i < SQ; ++i)
#pragma unroll
    for (int a = 0; a < TM; ++a) ssq[i][a] = 0.f;
  auto squares = [&](int h, int s) __attribute__((always_inline)) {
    if (sq_wn != s % WN) return;
#pragma unroll
    for (int a = 0; a < TM; ++a) {
      const uint4 v = __builtin_bit_cast(uint4, fa[h][a]);
      float t = ssq[s / WN][a];
      t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.x), __builtin_bit_cast(bf16x2, v.x), t, false);
      t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.y), __builtin_bit_cast(bf16x2, v.y), t, false);
      t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.z), __builtin_bit_cast(bf16x2, v.z), t, false);
      t = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v.w), __builtin_bit_cast(bf16x2, v.w), t, false);
      ssq[s / WN][a] = t;
    }
  };
  auto products = [&](int h) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
      for (int b = 0; b < TN; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[h][a], fb[h][b], acc[a][b], 0, 0, 0);
  };

  // the order of the loop: an activation slice, then a weight slice, then another
  load_w();
#pragma unroll
  for (int i = 0; i < STAGES - 1; ++i) {
    load_a();
    load_w();
    load_w();
  }
  wait_loads_and_meet<(STAGES - 1) * 2 * W_PER + (STAGES - 2) * A_PER>();
  fragments(0, 0);
  __builtin_amdgcn_s_waitcnt(0xc07f);  // LDS and scalar loads of the prologue: the loop's waits then count its own reads only
  // Half a slice: two k-steps.  The fragments of a k-step are requested one k-step ahead; the loads for the LDS that the
  // last meeting set free go out first; the next meeting comes while this half's last products are still to be issued.
  auto half_slice = [&](auto half_c, bool live) __attribute__((always_inline)) {
    constexpr int half = decltype(half_c)::value;
    fragments(1, half * 2 + 1);
    if (half == 0) load_a();
    load_w();
    __builtin_amdgcn_sched_barrier(0);
    if (live) {
      products(0);
      if (NORM) squares(0, half * 2);
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_loads_and_meet<(STAGES - 1) * 2 * W_PER + (STAGES - (half == 0 ? 1 : 2)) * A_PER>();
    w_cur = w_cur == (2 * STAGES - 1) * S::W_SLICE ? 0 : w_cur + S::W_SLICE;
    if (half == 1) a_cur = a_cur == (STAGES - 1) * S::A_SLICE ? 0 : a_cur + S::A_SLICE;
    fragments(0, half == 0 ? 2 : 0);
    __builtin_amdgcn_sched_barrier(0);
    if (live) {
      products(1);
      if (NORM) squares(1, half * 2 + 1);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int i = 0; i < rounds; ++i) {
    const bool live = KG == 1 || i < n;
    half_slice(std::integral_constant<int, 0>{}, live);
    half_slice(std::integral_constant<int, 1>{}, live);
  }
  wait_loads_and_meet<0>();  // nothing may land in LDS any more: the epilogue reuses it
  float *sS = reinterpret_cast<float *>(smem_all + S::sums), *chunk = sS + BM;  // chunk: [KG][BM][8]
  if (NORM) {
#pragma unroll
    for (int i = 0; i < SQ; ++i)
#pragma unroll
      for (int a = 0; a < TM; ++a)
        if (sq_wn + i * WN < 4) chunk[((kg * BM + (wm * TM + a) * 32 + ln) * 4 + sq_wn + i * WN) * 2 + lh] = ssq[i][a];
  }
  if (KG > 1 && kg > 0) {
    float *to = reinterpret_cast<float *>(smem_all) + ((kg - 1) * NW + wave) * (TM * TN * 1024) + lane * 4;
    static_for<TM * TN * 4>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value, t = i / 4, q = i % 4;
      const f32x16 &c = acc[t / TN][t % TN];
      *reinterpret_cast<f32x4 *>(to + i * 256) = f32x4{c[q * 4], c[q * 4 + 1], c[q * 4 + 2], c[q * 4 + 3]};
    });
  }
  if (NORM || KG > 1) __syncthreads();
  if (KG > 1 && kg > 0) return;  // a barrier counts the waves that are left
  if (KG > 1) {
#pragma unroll
    for (int g = 1; g < KG; ++g) {  // the groups' sums, in split order
      const float *from = reinterpret_cast<const float *>(smem_all) + ((g - 1) * NW + wave) * (TM * TN * 1024) + lane * 4;
      static_for<TM * TN * 4>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value, t = i / 4, q = i % 4;
        const f32x4 v = *reinterpret_cast<const f32x4 *>(from + i * 256);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) acc[t / TN][t % TN][q * 4 + e4] += v[e4];
      });
    }
  }
  if (NORM) {
    if (tid < BM) {
      float t = 0.f;
#pragma unroll
      for (int g = 0; g < KG; ++g) {
        const float *c = chunk + (g * BM + tid) * 8;
        t += ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
      }
      sS[tid] = t;
    }
    __syncthreads();
  }
  gemm_finish<TM, TN, NW, WM>(acc, e, M, N, KG == 1 ? split_k : 1, partial, tn, ks, m0, (tn * WN + wn) * TN, smem_all,
                              NORM ? sS : nullptr, ssq_part, K, eps);
#endif
}

// NORM_ALONE: a tile that runs with the fused norm only; the other form is not built
template <int WM, int WN, int TM, int TN, int STAGES, int KG = 1, bool NORM_ALONE = false>
hipError_t ensure_block_lds() {
  using S = BlockShape<WM, WN, TM, TN, STAGES, KG>;
  constexpr int cap = (int)S::lds;
  if (cap <= 64 * 1024) return hipSuccess;
  static bool raised[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (raised[dev]) return hipSuccess;
  auto raise = [](const void *f) { return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, cap); };
  hipError_t err = hipSuccess;
  if constexpr (!NORM_ALONE) err = raise(reinterpret_cast<const void *>(&gemm_block_kernel<WM, WN, TM, TN, STAGES, KG, 0>));
  if (err == hipSuccess) err = raise(reinterpret_cast<const void *>(&gemm_block_kernel<WM, WN, TM, TN, STAGES, KG, 1>));
  if (err == hipSuccess) raised[dev] = true;
  return err;
}

template <int WM, int WN, int TM, int TN, int STAGES, int KG = 1, bool NORM_ALONE = false>
hipError_t run_block(const GemmArgs &a, hipStream_t s, int split) {
  using S = BlockShape<WM, WN, TM, TN, STAGES, KG>;
  if (NORM_ALONE && !a.fused_norm) return hipErrorInvalidValue;
  const Plan p = make_plan(a.M, a.N, a.K, S::BM, S::BN, split);
  if (KG > 1 ? p.split_k != KG : !plan_fits(p, S::BM, a.ws, a.ws_bytes)) return hipErrorInvalidValue;
  const bool two = KG == 1 && p.split_k > 1;  // a second launch adds the partial tiles
  const int groups = (p.tiles_n * (KG > 1 ? 1 : p.split_k) + XCDS - 1) / XCDS;
  float *ssq_part = two ? (float *)a.ws : nullptr;
  float *partial = two ? (float *)((char *)a.ws + GEMM_SSQ_BYTES) : nullptr;
  if (a.am_val && (p.split_k != 1 || a.am_stride < p.tiles_n || a.fused_norm)) return hipErrorInvalidValue;
  if (a.am_val && a.am_parts_out) *a.am_parts_out = p.tiles_n;
  const Epilogue e = make_epilogue(a);
  const hipError_t set = ensure_block_lds<WM, WN, TM, TN, STAGES, KG, NORM_ALONE>();
  if (set != hipSuccess) return set;
  auto launch = [&](auto kernel) {
    kernel<<<groups * XCDS * p.tiles_m, 64 * S::NW * KG, S::lds, s>>>(
        (const bf16_t *)a.x, (const uint4 *)a.w, e, a.M, a.N, a.K, p.tiles_m, p.tiles_n, p.split_k, p.kt_per_split, partial,
        a.norm_eps, ssq_part);
  };
  if (a.fused_norm) launch(&gemm_block_kernel<WM, WN, TM, TN, STAGES, KG, 1>);
  if constexpr (!NORM_ALONE)
    if (!a.fused_norm) launch(&gemm_block_kernel<WM, WN, TM, TN, STAGES, KG, 0>);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || !two) return err;
  return launch_split_finish(partial, a.fused_norm ? ssq_part : nullptr, e, p.split_k, a, s);
}

}  // namespace
}  // namespace sf
