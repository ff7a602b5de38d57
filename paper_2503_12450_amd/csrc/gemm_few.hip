// Matrix products on few rows: C = A W^T with the epilogues of gemm.hip.
//
// A product of a few dozen or a few hundred rows is bound by latency: its
// tiles do not fill the chip, and a tile's time is its chain of K slices.
// What differs from the tiled kernel of gemm.hip:
//  * 16-row MFMAs, so a wave's tile can be as small as 16 x 16 and the tile
//    of a workgroup any multiple of 16: the launcher picks the shape that
//    spreads the outputs evenly over the CUs;
//  * the fragments of the next ring stage are read from LDS as a whole while
//    the current one multiplies, so a slice does not pay an LDS round trip
//    per k-step; reading them also frees their stage, which receives the
//    stage STAGES ahead at once (STAGES - 1 always in flight);
//  * the loads go out between the MFMAs;
//  * a tile of one wave needs no barrier at all;
//  * the epilogue's inputs (bias, residual, gate) are loaded before the main
//    loop, and results are stored from registers.
// What bounds a slice of the multi-wave tiles now is LDS bandwidth (128 bytes
// a cycle: a 64 x 64 tile's slice is 16 KiB written and 32 KiB read, 384
// cycles; measured 0.17 us), of the one-wave tile the issue of its loads.
// Measured on MI355X, the 64 x 64 tiles of the tiled kernel before and this
// after, weights from the Infinity Cache: 10 x 1024 x 1024 5.9 -> 3.1 us, 96
// x 768 x 3072 13.3 -> 6.0, 640 x 768 x 3072 14.1 -> 9.2, 512 x 1280 x 1280
// 7.7 -> 6.3, 1024 x 1536 x 1536 11.8 -> 9.0; fp32 80 x 768 x 3072 58.7 ->
// 25.7.  Deeper rings changed nothing; fragments loaded from memory straight
// into registers (16 rows x 64 bytes per load: one 16-byte request per cycle)
// were up to three times slower.
//
// Bits: v_mfma_f32_16x16x32_bf16 sums its 32 k as two v_mfma_f32_32x32x16_bf16
// in sequence do, and v_mfma_f32_16x16x4_f32 its 4 k as two
// v_mfma_f32_32x32x2_f32 do; with fp32 operands fed in the order of the tiled
// kernel (k 0, 4, 1, 5, 2, 6, 3, 7 of every eight), both kernels sum every
// output in the same order: the choice never changes a result bit.
#include <type_traits>
#include <utility>

#include "gemm_common.h"

namespace marcache {

namespace {

// One k-step: 64 bytes of K per row, lane -> row lane % 16, chunk lane / 16.
__device__ __forceinline__ void mma_step(f32x4_t& acc, const u32x4_t& w, const u32x4_t& a, bf16_t*) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, a), acc,
                                                0, 0, 0);
}
__device__ __forceinline__ void mma_step(f32x4_t& acc, const u32x4_t& w, const u32x4_t& a, float*) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[j]), __uint_as_float(a[j]), acc, 0, 0, 0);
}

// A fragment as read -> MFMA operands.  bf16: as read.  fp32: the four lane
// groups hold k 4 g .. 4 g + 3 of the step's sixteen; swapping the upper lanes
// of one register with the lower lanes of the next gives the operands k (0, 4,
// 1, 5), (2, 6, 3, 7), (8, 12, 9, 13), (10, 14, 11, 15).
__device__ __forceinline__ u32x4_t operand(const u32x4_t& v, bf16_t*) { return v; }
__device__ __forceinline__ u32x4_t operand(const u32x4_t& v, float*) {
  const auto s = __builtin_amdgcn_permlane32_swap(v[0], v[1], false, false);
  const auto t = __builtin_amdgcn_permlane32_swap(v[2], v[3], false, false);
  return u32x4_t{s[0], t[0], s[1], t[1]};
}

template <class F, int... I>
__device__ __forceinline__ void for_each_index(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}

// Workgroup of WM x WN waves, each 16 TM x 16 TN outputs.  The tile's rows of
// A, then of W, walk K through a ring of STAGES stages of U slices of 128
// bytes per row.
template <typename T, int TM, int TN, int WM, int WN, int U, int STAGES, int KIND>
__global__ __launch_bounds__(64 * WM * WN) void gemm_few_kernel(const T* __restrict__ A, const T* __restrict__ W,
                                                                int M, int N, int K, EpiArgs e) {
  constexpr bool kF32Out = KIND == EPI_RESIDUAL || KIND == EPI_GATE || sizeof(T) == 4;
  constexpr bool kResid = KIND == EPI_RESIDUAL || KIND == EPI_GATE;
  constexpr int ES = sizeof(T);
  constexpr int NW = WM * WN;
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN, ROWS = BM + BN;
  constexpr int SLICE_BYTES = ROWS * 128, STAGE_BYTES = U * SLICE_BYTES;
  constexpr int GROUPS = ROWS / 8;                     // wave-wide loads (8 rows, 1 KiB) per slice
  constexpr int LOADS = U * ((GROUPS + NW - 1) / NW);  // per wave and stage; a spare one repeats the last group
  constexpr int STEPS = 2 * U;                         // k-steps of 64 bytes per stage
  static_assert(STAGES >= 3 && (STAGES - 1) * LOADS < 64, "loads in flight");
  __shared__ __align__(1024) unsigned char ring[STAGES * STAGE_BYTES];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave - (wave / WN) * WN;
  const int lrow = lane & 15, lgrp = lane >> 4;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  int tm, tn;
  tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int Kb = __builtin_amdgcn_readfirstlane(K * ES);
  const int slices = Kb / 128;  // K * sizeof(T) is a multiple of 128
  const int KT = (slices + U - 1) / U;

  // The epilogue's inputs; acc[i][j][r] is row m_w + 16 i + lane % 16, column
  // n_w + 16 j + 4 (lane / 16) + r.  The output may be the residual itself:
  // each element is read here by the lane that writes it.
  const int m_w = m0 + wm * 16 * TM, n_w = n0 + wn * 16 * TN;
  u32x4_t bias[TN], res[TM][TN];
  u32x2_t gate[TM][TN];
  {
    const rsrc_t rb = make_out(const_cast<float*>(e.bias), static_cast<unsigned>(N) * 4u);
    const rsrc_t rr = make_out(kResid ? const_cast<float*>(e.resid) : nullptr,
                               kResid ? static_cast<unsigned>(M) * N * 4u : 0u);
    const rsrc_t rg = make_out(KIND == EPI_GATE ? const_cast<void*>(e.gate) : nullptr,
                               KIND == EPI_GATE ? static_cast<unsigned>(M) * e.gate_ld * ES : 0u);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n_w + 16 * j + 4 * lgrp;
      bias[j] = bload16(rb, n < N ? n * 4 : kOob);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int m = m_w + 16 * i + lrow;
        const bool ok = m < M && n < N;
        if constexpr (kResid) res[i][j] = bload16(rr, ok ? (m * N + n) * 4 : kOob);
        if constexpr (KIND == EPI_GATE)
          gate[i][j] = __builtin_amdgcn_raw_buffer_load_b64(rg, ok ? (m * e.gate_ld + n) * 2 : kOob, 0, 0);
      }
    }
  }

  // rows past M / N read as zeros
  const i32x4_t ra = make_rsrc(A + static_cast<long>(m0) * K, static_cast<unsigned>(min(BM, M - m0)) * Kb);
  const i32x4_t rw = make_rsrc(W + static_cast<long>(n0) * K, static_cast<unsigned>(min(BN, N - n0)) * Kb);
  const unsigned lds0 = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(
      static_cast<int>(reinterpret_cast<uintptr_t>(static_cast<unsigned char*>(ring)))));
  // Group q holds rows 8 q .. 8 q + 7: lane -> row lane / 8, chunk lane % 8,
  // which is the row's chunk (lane % 8) ^ (row / 2) % 8 (16 rows of one chunk
  // then fall on all 64 banks): one lane offset for even, one for odd groups
  const int g_row = lane >> 3, g_ch = lane & 7;
  // (the offsets differ in bit 6: Kb is a multiple of 128).
  const int voff0 = g_row * Kb + ((g_ch ^ (g_row >> 1)) << 4);
  // load l of stage kt of K into ring stage `to`; slices past the end repeat
  // the last one (and are not multiplied)
  auto issue = [&](int to, int kt, int l) {
    const int u = l % U;
    const int q = min(wave + NW * (l / U), GROUPS - 1);
    const unsigned dst = lds0 + to * STAGE_BYTES + u * SLICE_BYTES + q * 1024;
    const bool is_a = q < BM / 8;
    i32x4_t r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r[c] = is_a ? ra[c] : rw[c];
    const int row = is_a ? 8 * q : 8 * q - BM;
    dma16(r, dst, voff0 ^ ((q & 1) << 6), min(kt * U + u, slices - 1) * 128 + row * Kb);
  };
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
#pragma unroll
    for (int l = 0; l < LOADS; ++l) issue(s, s, l);

  // fragments: lane -> row lane % 16 of a 16-row tile, chunk 4 s + lane / 16
  // of k-step s
  const int sw = (lrow >> 1) & 7;
  int a_off[2], w_off[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    a_off[s] = (wm * 16 * TM + lrow) * 128 + (((4 * s + lgrp) ^ sw) << 4);
    w_off[s] = (BM + wn * 16 * TN + lrow) * 128 + (((4 * s + lgrp) ^ sw) << 4);
  }
  struct Frags {
    u32x4_t a[STEPS][TM], w[STEPS][TN];
  };
  auto read = [&](Frags& f, int from) {
    const unsigned char* base = ring + from * STAGE_BYTES;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
        f.w[s][j] = *reinterpret_cast<const u32x4_t*>(base + (s / 2) * SLICE_BYTES + w_off[s & 1] + j * 2048);
#pragma unroll
      for (int i = 0; i < TM; ++i)
        f.a[s][i] = *reinterpret_cast<const u32x4_t*>(base + (s / 2) * SLICE_BYTES + a_off[s & 1] + i * 2048);
    }
  };
  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // k-steps [s0, s1) of a stage's fragments; with LOAD, the stage's loads go
  // out between the MFMAs (issued in a row they hold the wave up: about 27
  // cycles each)
  auto multiply = [&](const Frags& f, int s0, int s1, auto load, int to, int kt) {
    constexpr bool LOAD = decltype(load)::value;
    constexpr int MMAS = STEPS * TM * TN;
    int done = 0;
#pragma unroll
    for (int s = s0; s < s1; ++s) {
      u32x4_t oa[TM], ow[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) oa[i] = operand(f.a[s][i], static_cast<T*>(nullptr));
#pragma unroll
      for (int j = 0; j < TN; ++j) ow[j] = operand(f.w[s][j], static_cast<T*>(nullptr));
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          mma_step(acc[i][j], ow[j], oa[i], static_cast<T*>(nullptr));
          if constexpr (LOAD) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int l = done * LOADS / MMAS; l < (done + 1) * LOADS / MMAS; ++l) issue(to, kt, l);
            __builtin_amdgcn_sched_barrier(0);
          }
          ++done;
        }
    }
  };
  // this wave's reads of the current slice have arrived and, past the
  // barrier, every wave's loads of the next slice and reads of this one
  auto sync = [&]() {
    if constexpr (NW > 1) lds_barrier();
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  };

  Frags f[2];
  wait_vm<(STAGES - 1) * LOADS>();
  sync();
  read(f[0], 0);
  // One stage: cur holds its fragments, nxt receives the next one's.
  int stage = 0;  // of cur
  auto advance = [&]() { stage = stage == STAGES - 1 ? 0 : stage + 1; };
  auto step = [&](Frags& cur, Frags& nxt, int kt) {
    wait_vm<(STAGES - 2) * LOADS>();
    sync();
    const int freed = stage;
    advance();
    read(nxt, stage);
    __builtin_amdgcn_sched_barrier(0);
    multiply(cur, 0, STEPS, std::true_type(), freed, kt + STAGES);
    __builtin_amdgcn_sched_barrier(0);
  };
  int kt = 0;
  for (; kt + 1 < KT - STAGES; kt += 2) {
    step(f[0], f[1], kt);
    step(f[1], f[0], kt + 1);
  }
  if (kt < KT - STAGES) {
    step(f[0], f[1], kt);
    f[0] = f[1];
  }
  // the last STAGES stages (fewer when K is short): nothing more to load
  auto tail = [&](auto index) {
    constexpr int j = decltype(index)::value;
    if (KT - STAGES + j < 0) return;
    Frags& cur = f[j & 1];
    Frags& nxt = f[(j & 1) ^ 1];
    if constexpr (j & 1)
      if (KT - STAGES + j == 0) cur = nxt;  // short K enters here, with its first stage in f[0]
    if constexpr (j < STAGES - 1) {
      wait_vm<(STAGES - 2 - j) * LOADS>();
      sync();
      advance();
      read(nxt, stage);
      __builtin_amdgcn_sched_barrier(0);
      multiply(cur, 0, STEPS, std::false_type(), 0, 0);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)  // the last stage may hold fewer slices
        if (u == 0 || (KT - 1) * U + u < slices) multiply(cur, 2 * u, 2 * u + 2, std::false_type(), 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  for_each_index(tail, std::make_integer_sequence<int, STAGES>());
  wait_vm<0>();  // no load may still target this workgroup's LDS

  // epilogue: four consecutive columns of one row per lane and tile; stores
  // past M or N fall outside the descriptors
  rsrc_t out, aux0, aux1, aux2;
  if constexpr (KIND == EPI_QKV) {
    const unsigned slots = static_cast<unsigned>((M + e.per_slot - 1) / e.per_slot);
    const unsigned cache = slots * e.n_heads * e.seq * e.d_head * ES;
    out = make_out(e.out, e.out ? static_cast<unsigned>(M) * e.d_model * ES : 0u);
    aux0 = make_out(e.k_cache, e.k_cache ? cache : 0u);
    aux1 = make_out(e.v_cache, e.v_cache ? cache : 0u);
    aux2 = make_out(e.v_copy, e.v_copy ? cache : 0u);
  } else {
    const unsigned rows = KIND == EPI_RESIDUAL && e.out_idx
                              ? static_cast<unsigned>((M + e.per_slot - 1) / e.per_slot) * e.seq
                              : static_cast<unsigned>(M);
    out = make_out(e.out, rows * N * (kF32Out ? 4u : 2u));
    aux0 = make_out(KIND == EPI_RESIDUAL ? e.resid_copy : nullptr,
                    KIND == EPI_RESIDUAL && e.resid_copy ? static_cast<unsigned>(M) * N * 4u : 0u);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m_w + 16 * i + lrow;
    const int mc = min(m, M - 1);
    int slot = 0, tok = 0, orow = mc;
    if constexpr (KIND == EPI_QKV) {
      slot = div_by(mc, e.slot_magic, e.slot_shift);
      tok = e.idx ? e.idx[mc] : mc - slot * e.per_slot;
    } else if constexpr (KIND == EPI_RESIDUAL) {
      if (e.out_idx) orow = div_by(mc, e.slot_magic, e.slot_shift) * e.seq + e.out_idx[mc];
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n_w + 16 * j + 4 * lgrp;
      const bool ok = m < M && n < N;
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[r] = acc[i][j][r] + __uint_as_float(bias[j][r]);
        if constexpr (KIND == EPI_GELU) x[r] = ES == 2 ? gelu_erf_bf16(x[r]) : gelu_erf(x[r]);
        if constexpr (KIND == EPI_SILU) x[r] = silu_f(x[r]);
        if constexpr (KIND == EPI_RESIDUAL) x[r] = __uint_as_float(res[i][j][r]) + x[r];
        if constexpr (KIND == EPI_GATE) {
          const uint32_t gw = gate[i][j][r >> 1];
          x[r] = fmaf(__uint_as_float((r & 1) ? (gw & 0xFFFF0000u) : (gw << 16)), x[r], __uint_as_float(res[i][j][r]));
        }
      }
      const u32x4_t v4 = {__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
      const u32x2_t v2 = {pack2bf(x[0], x[1]), pack2bf(x[2], x[3])};
      auto put = [&](rsrc_t r, int elem, bool valid) {
        if constexpr (kF32Out) __builtin_amdgcn_raw_buffer_store_b128(v4, r, valid ? elem * 4 : kOob, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(v2, r, valid ? elem * 2 : kOob, 0, 0);
      };
      if constexpr (KIND == EPI_QKV) {
        const int ng = n + e.n_offset;
        const int sec = qkv_section(e, ng);
        const int col = ng - sec * e.d_model;  // head * d_head + d
        const int head = div_by(col, e.head_magic, e.head_shift);
        const int at = ((slot * e.n_heads + head) * e.seq + tok) * e.d_head + (col - head * e.d_head);
        put(out, mc * e.d_model + col, ok && sec == 0);
        put(aux0, at, ok && sec == 1);
        put(aux1, at, ok && sec == 2);
        if (e.v_copy) put(aux2, at, ok && sec == 2);
      } else {
        put(out, orow * N + n, ok);
        if constexpr (KIND == EPI_RESIDUAL)
          if (e.resid_copy) put(aux0, mc * N + n, ok);
      }
    }
  }
}

template <typename T, int TM, int TN, int WM, int WN, int U, int STAGES, int KIND>
hipError_t few_as(const void* A, const void* W, int M, int N, int K, const EpiArgs& e, hipStream_t st) {
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
  const int tiles = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  auto kern = gemm_few_kernel<T, TM, TN, WM, WN, U, STAGES, KIND>;
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(64 * WM * WN), 0, st, static_cast<const T*>(A), static_cast<const T*>(W),
                     M, N, K, e);
  return hipGetLastError();
}

template <typename T, int KIND>
hipError_t few_pick(int tile, const void* A, const void* W, int M, int N, int K, const EpiArgs& e, hipStream_t st) {
  switch (tile) {
    case FEW_16x16: return few_as<T, 1, 1, 1, 1, 2, 5, KIND>(A, W, M, N, K, e, st);
    case FEW_32x32: return few_as<T, 1, 1, 2, 2, 2, 5, KIND>(A, W, M, N, K, e, st);
    case FEW_32x64: return few_as<T, 1, 2, 2, 2, 2, 4, KIND>(A, W, M, N, K, e, st);
    case FEW_64x48: return few_as<T, 1, 3, 4, 1, 2, 4, KIND>(A, W, M, N, K, e, st);
    default: break;
  }
  // fp32 is bound by its MFMAs from here on and stays with the tiled kernel
  if constexpr (sizeof(T) == 4) return hipErrorInvalidValue;
  else switch (tile) {
    case FEW_64x64: return few_as<T, 2, 2, 2, 2, 1, 5, KIND>(A, W, M, N, K, e, st);
    case FEW_64x96: return few_as<T, 2, 3, 2, 2, 1, 5, KIND>(A, W, M, N, K, e, st);
    case FEW_128x64: return few_as<T, 4, 2, 2, 2, 1, 5, KIND>(A, W, M, N, K, e, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t few_kind(int tile, const void* A, const void* W, int M, int N, int K, const EpiArgs& e, hipStream_t st) {
  switch (e.kind) {
    case EPI_BIAS: return few_pick<T, EPI_BIAS>(tile, A, W, M, N, K, e, st);
    case EPI_GELU: return few_pick<T, EPI_GELU>(tile, A, W, M, N, K, e, st);
    case EPI_RESIDUAL: return few_pick<T, EPI_RESIDUAL>(tile, A, W, M, N, K, e, st);
    case EPI_QKV: return few_pick<T, EPI_QKV>(tile, A, W, M, N, K, e, st);
    default: break;
  }
  if constexpr (sizeof(T) == 2) {
    switch (e.kind) {
      case EPI_SILU: return few_pick<T, EPI_SILU>(tile, A, W, M, N, K, e, st);
      case EPI_GATE: return few_pick<T, EPI_GATE>(tile, A, W, M, N, K, e, st);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_few(int dtype, int tile, const void* A, const void* W, int M, int N, int K, const EpiArgs& e,
                           hipStream_t st) {
  if (dtype == DT_BF16) return few_kind<bf16_t>(tile, A, W, M, N, K, e, st);
  return few_kind<float>(tile, A, W, M, N, K, e, st);
}

}  // namespace marcache
