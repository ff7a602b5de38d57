// MAR's per-token diffusion head with classifier-free guidance (the
// condition cache's unconditional rows feed its unconditional branch): the
// network, the DDPM sampler and their C ABI (include/mar_head.h).
//
// One call samples R tokens.  The conditional and the unconditional
// evaluation of every token run as one batch of 2R rows (rows [0, R)
// conditional, [R, 2R) unconditional), so each product of the network is
// one launch over 2R rows:
//   per call           gather z rows -> bf16; c = z W_z^T + b_z (fp32)
//   per C sampling     s = silu(c + e_i) (bf16), C steps' rows
//   steps              m = s W_ada^T + b_ada (every block's shift/scale/gate
//                          and the final shift/scale, of C steps in one
//                          product: s depends neither on the block nor on x)
//   per sampling step  per block: u = ln(h)(1 + scale) + shift (bf16);
//                          g = silu(u W1^T + b1) (bf16);
//                          h = h + gate (g W2^T + b2) (fp32, in place)
//                      step: per token, both rows' final ln-modulation and
//                          output product, the guidance mix, the DDPM update
//                          of the token's latent x, then the next step's h =
//                          x W_in^T + b_in and its first block's u
// The products are the block GEMM kernels with the SILU and GATE epilogues.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <memory>
#include <mutex>
#include <new>
#include <system_error>

#include "../../include/mar_head.h"
#include "gemm_common.h"

using namespace marcache;

namespace {

mar_status hfail(mar_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  abi_fail_v(s, fmt, ap);
  va_end(ap);
  return s;
}

#define HEAD_HIP(call, what)                                                          \
  do {                                                                                \
    hipError_t e_ = (call);                                                           \
    if (e_ != hipSuccess) return hfail(MAR_E_DEVICE, "%s: %s", what, hipGetErrorString(e_)); \
  } while (0)

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------

// The respaced DDPM coefficients of every sampling step i, in fp64 on one
// thread (a running product over the training steps): coef[i] = (1 /
// sqrt(1 - beta_i), beta_i / sqrt(1 - abar_i), sigma_i, t_i), with t_i =
// floor(i * train_steps / steps), abar_i the product of (1 - beta) up to
// t_i, beta_i = 1 - abar_i / abar_(i-1), sigma_i^2 = beta_i (1 - abar_(i-1))
// / (1 - abar_i) and sigma_0 = 0.
__global__ void head_schedule_kernel(int steps, int train_steps, double beta_start, double beta_end,
                                     f32x4_t* __restrict__ coef) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double step = train_steps > 1 ? (beta_end - beta_start) / (train_steps - 1) : 0.0;
  double abar = 1.0, abar_kept = 1.0;
  int next = 0;
  for (int k = 0; k < train_steps && next < steps; ++k) {
    abar *= 1.0 - (beta_start + step * k);
    while (next < steps && static_cast<long>(next) * train_steps / steps == k) {
      const double beta = 1.0 - abar / abar_kept;
      const double sigma = next == 0 ? 0.0 : sqrt(beta * (1.0 - abar_kept) / (1.0 - abar));
      coef[next] = f32x4_t{static_cast<float>(1.0 / sqrt(1.0 - beta)), static_cast<float>(beta / sqrt(1.0 - abar)),
                           static_cast<float>(sigma), static_cast<float>(k)};
      abar_kept = abar;
      ++next;
    }
  }
}

// Sinusoidal features of every sampling step's timestep, bf16 [steps, F]:
// [cos(t f_k) for k < F/2, sin(t f_k) ...], f_k = 10000^(-k / (F/2)), in
// fp64 before the rounding.
__global__ void head_phi_kernel(const f32x4_t* __restrict__ coef, int steps, int F, bf16_t* __restrict__ phi) {
  const int i = blockIdx.x;
  const int half = F / 2;
  if (i >= steps) return;
  const double t = coef[i][3];
  for (int k = threadIdx.x; k < F; k += blockDim.x) {
    const int j = k < half ? k : k - half;
    const double a = t * exp(-log(10000.0) * j / half);
    phi[static_cast<long>(i) * F + k] = f2bf(static_cast<float>(k < half ? cos(a) : sin(a)));
  }
}

__global__ void head_fill_zero_kernel(float* __restrict__ p, long n4) {
  const long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n4) reinterpret_cast<f32x4_t*>(p)[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// Rows [0, R) of `out` from y_cond[row_cond[r]], rows [R, 2R) from
// y_uncond[row_uncond[r]], rounded to bf16; an index outside [0, y_rows)
// gives a zero row.  One wave per output row.
__global__ __launch_bounds__(256) void head_gather_kernel(const float* __restrict__ yc,
                                                          const float* __restrict__ yu, int y_rows,
                                                          const int32_t* __restrict__ rc,
                                                          const int32_t* __restrict__ ru, int R, int D,
                                                          bf16_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= 2 * R) return;
  const bool unc = row >= R;
  const int r = unc ? row - R : row;
  const int src = unc ? ru[r] : rc[r];
  const float* y = unc ? yu : yc;
  const bool ok = src >= 0 && src < y_rows;
  for (int c = lane * 4; c < D; c += 256) {
    f32x4_t v = ok ? *reinterpret_cast<const f32x4_t*>(y + static_cast<long>(src) * D + c) : f32x4_t{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<u32x2_t*>(out + static_cast<long>(row) * D + c) = u32x2_t{pack2bf(v[0], v[1]), pack2bf(v[2], v[3])};
  }
}

__device__ __forceinline__ float silu_h(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

// in_w [w, T] -> in_wt [T, w] (bf16), once at init, so that a lane reads four
// consecutive columns of one input component per load.
__global__ void head_transpose_in_kernel(const bf16_t* __restrict__ in_w, int w, int T, bf16_t* __restrict__ in_wt) {
  const long i = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= static_cast<long>(w) * T) return;
  const int col = static_cast<int>(i / T), j = static_cast<int>(i - static_cast<long>(col) * T);
  in_wt[static_cast<long>(j) * w + col] = in_w[i];
}

// s[k 2R + r] = silu(c[r] + e[i0 - k]) (bf16) for the 2R rows of every of C
// sampling steps i0, i0 - 1, ..., one wave per row.
__global__ __launch_bounds__(256) void head_silu_kernel(const float* __restrict__ c, const float* __restrict__ e,
                                                        int i0, int C, int R2, int w, bf16_t* __restrict__ s) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= C * R2) return;
  const int k = row / R2;
  const float* cr = c + static_cast<long>(row - k * R2) * w;
  const float* er = e + static_cast<long>(i0 - k) * w;
  bf16_t* sr = s + static_cast<long>(row) * w;
  for (int col = lane * 4; col < w; col += 256) {
    const f32x4_t cv = *reinterpret_cast<const f32x4_t*>(cr + col);
    const f32x4_t ev = *reinterpret_cast<const f32x4_t*>(er + col);
    *reinterpret_cast<u32x2_t*>(sr + col) =
        u32x2_t{pack2bf(silu_h(cv[0] + ev[0]), silu_h(cv[1] + ev[1])), pack2bf(silu_h(cv[2] + ev[2]), silu_h(cv[3] + ev[3]))};
  }
}

// Rows of the head are held 4 columns per lane per group: group k of lane
// l is columns 4 l + 256 k .. + 3.  EXACT: the width is exactly 256 G, so
// no group needs a bounds check (1024, 1280, 1536 = 256 x 4, 5, 6);
// otherwise groups past the width are skipped.
template <int G, bool EXACT>
__device__ __forceinline__ bool group_in(int lane, int k, int w) {
  return EXACT || lane * 4 + 256 * k < w;
}

__device__ __forceinline__ float bf_lo(uint32_t a) { return __uint_as_float(a << 16); }
__device__ __forceinline__ float bf_hi(uint32_t a) { return __uint_as_float(a & 0xFFFF0000u); }

// Row statistics (mean, 1 / sqrt(var + eps)) of a row held in v, with in(k)
// for the groups that this lane has, summed per lane in column order and then
// across the wave: the step kernel's waves hold a row in the same way, so both
// give the same bits.
template <int G, class In>
__device__ __forceinline__ void row_stats(const f32x4_t (&v)[G], In&& in, int w, float eps, float& mean, float& rstd) {
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < G; ++k)
    if (in(k)) sum += (v[k][0] + v[k][1]) + (v[k][2] + v[k][3]);
  mean = wave_sum(sum) / static_cast<float>(w);
  float sq = 0.f;
#pragma unroll
  for (int k = 0; k < G; ++k)
    if (in(k))
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float d = v[k][q] - mean;
        sq = fmaf(d, d, sq);
      }
  rstd = __builtin_amdgcn_rsqf(wave_sum(sq) / static_cast<float>(w) + eps);
}

// Four values of a row: (v - mean) rstd (1 + scale) + shift.
__device__ __forceinline__ void mod4(f32x4_t& v, float mean, float rstd, const u32x2_t& sh, const u32x2_t& sc) {
  v[0] = fmaf((v[0] - mean) * rstd, 1.0f + bf_lo(sc[0]), bf_lo(sh[0]));
  v[1] = fmaf((v[1] - mean) * rstd, 1.0f + bf_hi(sc[0]), bf_hi(sh[0]));
  v[2] = fmaf((v[2] - mean) * rstd, 1.0f + bf_lo(sc[1]), bf_lo(sh[1]));
  v[3] = fmaf((v[3] - mean) * rstd, 1.0f + bf_hi(sc[1]), bf_hi(sh[1]));
}

// v <- ln(v) (1 + scale) + shift for row `row` of h, with the shift and
// scale at columns shift_off / scale_off of the modulation row mr.  Every
// load (the row, then the shift and scale) is issued before the first
// reduction.
template <int G, bool EXACT>
__device__ __forceinline__ void load_lnmod(const float* __restrict__ hrow, const bf16_t* __restrict__ mr,
                                           int shift_off, int scale_off, int lane, int w, float eps,
                                           f32x4_t (&v)[G]) {
  u32x2_t sh[G], sc[G];
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const int col = lane * 4 + 256 * k;
    if (group_in<G, EXACT>(lane, k, w)) {
      v[k] = *reinterpret_cast<const f32x4_t*>(hrow + col);
      sh[k] = *reinterpret_cast<const u32x2_t*>(mr + shift_off + col);
      sc[k] = *reinterpret_cast<const u32x2_t*>(mr + scale_off + col);
    } else {
      v[k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      sh[k] = sc[k] = u32x2_t{0u, 0u};
    }
  }
  float mean, rstd;
  row_stats(v, [&](int k) { return group_in<G, EXACT>(lane, k, w); }, w, eps, mean, rstd);
#pragma unroll
  for (int k = 0; k < G; ++k) mod4(v[k], mean, rstd, sh[k], sc[k]);
}

// u[r] = ln(h[r]) (1 + scale[r]) + shift[r] (bf16), one wave per row; the
// shift and scale are columns [shift_off, +w) and [scale_off, +w) of the
// modulation rows m [rows, ld] (bf16).
template <int G, bool EXACT>
__global__ __launch_bounds__(256) void head_lnmod_kernel(const float* __restrict__ h,
                                                         const bf16_t* __restrict__ m, int ld, int shift_off,
                                                         int scale_off, int rows, int w, float eps,
                                                         bf16_t* __restrict__ u) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const long base = static_cast<long>(row) * w;
  f32x4_t v[G];
  load_lnmod<G, EXACT>(h + base, m + static_cast<long>(row) * ld, shift_off, scale_off, lane, w, eps, v);
#pragma unroll
  for (int k = 0; k < G; ++k) {
    const int col = lane * 4 + 256 * k;
    if (group_in<G, EXACT>(lane, k, w))
      *reinterpret_cast<u32x2_t*>(u + base + col) = u32x2_t{pack2bf(v[k][0], v[k][1]), pack2bf(v[k][2], v[k][3])};
  }
}

// The end of a sampling step and the start of the next, one workgroup per
// token r: part p of it (nwr waves) has row r + p R (p = 0 the conditional
// row, 1 the unconditional one).  A row is GT groups of 256 columns at most,
// 4 per lane; a wave loads and stores OWN of them.
//  out   the row's final ln-modulation and output product; then the guided
//        prediction eps = eps_u + scale (eps_c - eps_u) and the DDPM update of
//        x[r] with the coefficients of sampling step i and the draw xi_i[r]
//        (not read when sigma_i = 0)
//  next  h = W_in x + b_in of the next step (x from memory without `out`)
//  u     the first block's u = ln(h)(1 + scale) + shift from the next step's
//        modulation rows
// What bounds it is latency: a chain of loads, four row sums and the sum of
// the output components.  So the loads are spread over the waves of a row and
// meet in LDS, and every wave then holds the whole row: it forms the
// statistics by itself (no exchange of partial sums) and a share of the output
// components; the weights of both products are loaded ahead of the reductions.
// As three kernels (one wave per row and 16 components; the prologue of the
// next step; the first ln-modulation) it took 12.6 + 8.7 + 3.6 us at 256 tokens
// of width 1280 on MI355X, as one 9.6.  Whole calls of ten sampling steps and two blocks,
// as three kernels and as this one: 5 tokens of width 1024 485 and 227 us, 64
// tokens of width 1024 and 64 components 1364 and 354 us, 256 tokens of width
// 1280 816 and 578 us.
//
// The order of every sum is that of one wave per row: a lane's columns in
// ascending order, then a fixed tree across the lanes.  With T <= 16 a wave
// forms C components: halving exchanges (lane distance 32, 16, ...) each keep
// half of the components and add the partner's copy of that half, until one is
// left; full exchanges complete the sum, leaving component o = the lane's
// upper bits in every lane of its group of 64 / C.  Wider tokens take one wave
// reduction per component.
struct StepArgs {
  const bf16_t *out_w, *in_wt, *m_out, *m_next;  // modulation rows of this and of the next step
  const float *out_b, *in_b, *xi;
  const f32x4_t* coef;
  float *h, *x, *traj, *eps_out;
  bf16_t* u;
  int ld, shift_out, scale_out;  // row stride of the modulation, the final shift and scale in it
  int i, R, w, T, nwr;
  float eps_ln, scale;
  int out, next;
};

template <int GT, int C>
__global__ __launch_bounds__(128 * (GT < 8 ? GT : 8)) void head_step_kernel(StepArgs a) {
  constexpr int TB = 16;                // components held in registers
  constexpr int OWN = GT > 8 ? 2 : 1;
  // Weights held ahead of the reductions: as many as the registers of a
  // workgroup of this many waves take (128 per lane at 14 and 16 waves).  Both
  // products' held past width 2048 spilled 46 to 173 registers to scratch
  // memory, which the runtime may have to allocate at the first launch; ten
  // steps of 5 tokens of width 4096 took 825 to 900 us that way, 735 this way.
  constexpr bool WV = GT <= 8, IV = GT <= 6;
  __shared__ f32x4_t row_v[2][GT][64];
  __shared__ u32x2_t row_sh[2][GT][64], row_sc[2][GT][64];
  __shared__ float eps[2][64];
  __shared__ float xs[64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwr = OWN == 1 ? GT : a.nwr, w = a.w, T = a.T;
  const int p = wave / nwr, wr = wave - p * nwr;
  const int r = blockIdx.x;
  const long row = r + static_cast<long>(p) * a.R;
  const int groups = OWN == 1 ? GT : (w + 255) / 256;
  // this lane's columns in group k of the row
  auto in_row = [&](int k) { return (OWN == 1 && k < GT - 1) || k * 256 + lane * 4 < w; };
  int col[OWN];
#pragma unroll
  for (int g = 0; g < OWN; ++g) col[g] = (wr + g * nwr) * 256 + lane * 4;
  // Loads through descriptors that end with the row (the matrix), of no bytes
  // where there is nothing to load: what lies past them reads as zeros, with
  // no branch around a load.
  auto load2 = [&](rsrc_t q, int at) { return __builtin_amdgcn_raw_buffer_load_b64(q, at, 0, 0); };
  auto load4 = [&](rsrc_t q, int at) { return __builtin_bit_cast(f32x4_t, bload16(q, at)); };
  const unsigned row4 = static_cast<unsigned>(w) * 4u, row2 = static_cast<unsigned>(w) * 2u;
  const rsrc_t r_h = make_out(a.h + row * w, row4);
  const rsrc_t r_ow = make_out(const_cast<bf16_t*>(a.out_w), a.out ? T * row2 : 0u);
  const rsrc_t r_iw = make_out(const_cast<bf16_t*>(a.in_wt), a.next ? T * row2 : 0u);
  // the whole row as the waves of this part have put it into LDS
  auto gather = [&](f32x4_t (&v)[GT]) {
#pragma unroll
    for (int k = 0; k < GT; ++k) v[k] = k < groups ? row_v[p][k][lane] : f32x4_t{0.f, 0.f, 0.f, 0.f};
  };

  // the loads of the kernel, ahead of the first reduction
  const int t0 = wr * C;  // this wave's first output component, with T <= TB
  const bool makes = a.out && t0 < T;
  const bool updates = wave == 0 && lane < T;
  const long at = static_cast<long>(r) * T + lane;
  float xv = 0.f, ob = 0.f, draw = 0.f;
  f32x4_t cf = {0.f, 0.f, 0.f, 0.f}, hv[OWN], hb[OWN];
  u32x2_t sh[OWN], sc[OWN], sh2[OWN], sc2[OWN], wv[WV ? C : 1][WV ? GT : 1], iv[TB][OWN];
  if (a.out) {
    const rsrc_t r_sh = make_out(const_cast<bf16_t*>(a.m_out) + row * a.ld + a.shift_out, row2);
    const rsrc_t r_sc = make_out(const_cast<bf16_t*>(a.m_out) + row * a.ld + a.scale_out, row2);
#pragma unroll
    for (int g = 0; g < OWN; ++g) {
      hv[g] = load4(r_h, col[g] * 4);
      sh[g] = load2(r_sh, col[g] * 2);
      sc[g] = load2(r_sc, col[g] * 2);
    }
  }
  if (updates) {
    xv = a.x[at];
    if (a.out) {
      cf = a.coef[a.i];
      ob = a.out_b[lane];
      if (a.i > 0) draw = a.xi[static_cast<long>(a.i) * a.R * T + at];  // sigma_0 = 0: entry 0 is not read
    }
  }
  auto out_weight = [&](int c, int k) {  // component t0 + c, group k
    return load2(r_ow, in_row(k) ? ((t0 + c) * w + k * 256 + lane * 4) * 2 : kOob);
  };
  if constexpr (WV) {
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int k = 0; k < GT; ++k) wv[c][k] = out_weight(c, k);
  }
  {
    const rsrc_t r_b = make_out(const_cast<float*>(a.in_b), a.next ? row4 : 0u);
    const rsrc_t r_m = make_out(const_cast<bf16_t*>(a.m_next) + row * a.ld, a.next && a.m_next ? 2 * row2 : 0u);
#pragma unroll
    for (int g = 0; g < OWN; ++g) {
      hb[g] = load4(r_b, col[g] * 4);
      sh2[g] = load2(r_m, col[g] * 2);  // (past the row only into the scale, in lanes that store nothing)
      sc2[g] = load2(r_m, (w + col[g]) * 2);
    }
  }
  auto in_weight = [&](int t, int g) { return load2(r_iw, col[g] < w ? (t * w + col[g]) * 2 : kOob); };
  auto load_in = [&]() {
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int g = 0; g < OWN; ++g) iv[t][g] = in_weight(t, g);
  };
  if constexpr (IV) load_in();
  if (a.out) {
#pragma unroll
    for (int g = 0; g < OWN; ++g) {
      row_v[p][wr + g * nwr][lane] = hv[g];
      row_sh[p][wr + g * nwr][lane] = sh[g];
      row_sc[p][wr + g * nwr][lane] = sc[g];
    }
    __syncthreads();
    if (T > TB || makes) {
      f32x4_t v[GT];
      gather(v);
      float mean, rstd;
      row_stats(v, in_row, w, a.eps_ln, mean, rstd);
#pragma unroll
      for (int k = 0; k < GT; ++k)
        if (k < groups) mod4(v[k], mean, rstd, row_sh[p][k][lane], row_sc[p][k][lane]);
      auto dot = [&](float s, const f32x4_t& x, const u32x2_t& q) {
        s = fmaf(x[0], bf_lo(q[0]), s);
        s = fmaf(x[1], bf_hi(q[0]), s);
        s = fmaf(x[2], bf_lo(q[1]), s);
        return fmaf(x[3], bf_hi(q[1]), s);
      };
      if (T <= TB) {
        float acc[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          float s = 0.f;
#pragma unroll
          for (int k = 0; k < GT; ++k)
            if (k < groups) s = dot(s, v[k], WV ? wv[WV ? c : 0][WV ? k : 0] : out_weight(c, k));
          acc[c] = s;
        }
        // reduce-scatter: after the exchange at distance d, lanes with that
        // bit set hold the upper half of the remaining components
#pragma unroll
        for (int half = C / 2, d = 32; half >= 1; half >>= 1, d >>= 1) {
          // (bit selects: written with ?: the compiler turns the picks into
          // dynamic indexes of acc, some 50 instructions each)
          const uint32_t up = (lane & d) != 0 ? ~0u : 0u;
          auto pick = [&](float a, float b) {
            return __uint_as_float((__float_as_uint(b) & up) | (__float_as_uint(a) & ~up));
          };
#pragma unroll
          for (int k = 0; k < half; ++k)
            acc[k] = pick(acc[k], acc[k + half]) + __shfl_xor(pick(acc[k + half], acc[k]), d, 64);
        }
        float tot = acc[0];
#pragma unroll
        for (int d = 32 / C; d >= 1; d >>= 1) tot += __shfl_xor(tot, d, 64);
        if (lane % (64 / C) == 0) eps[p][t0 + lane / (64 / C)] = tot;
      } else {
        for (int t = wr; t < T; t += nwr) {
          float s = 0.f;
#pragma unroll
          for (int k = 0; k < GT; ++k)
            if (in_row(k)) s = dot(s, v[k], load2(r_ow, (t * w + k * 256 + lane * 4) * 2));
          const float tot = wave_sum(s);
          if (lane == 0) eps[p][t] = tot;
        }
      }
    }
    if constexpr (!IV) load_in();
    __syncthreads();
    if (updates) {
      const float ec = eps[0][lane] + ob, eu = eps[1][lane] + ob;
      const float eg = fmaf(a.scale, ec - eu, eu);
      xv = cf[0] * fmaf(-cf[1], eg, xv);
      if (cf[2] != 0.f) xv = fmaf(cf[2], draw, xv);
      a.x[at] = xv;
      if (a.traj) a.traj[at] = xv;
      if (a.eps_out) a.eps_out[at] = eg;
    }
  }
  if (!a.next) return;
  if (!IV && !a.out) load_in();
  if (wave == 0) xs[lane] = xv;  // zeros past T
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TB; ++j) {  // the weights past T are zeros
    const float xj = xs[j];
#pragma unroll
    for (int g = 0; g < OWN; ++g) {
      hb[g][0] = fmaf(xj, bf_lo(iv[j][g][0]), hb[g][0]);
      hb[g][1] = fmaf(xj, bf_hi(iv[j][g][0]), hb[g][1]);
      hb[g][2] = fmaf(xj, bf_lo(iv[j][g][1]), hb[g][2]);
      hb[g][3] = fmaf(xj, bf_hi(iv[j][g][1]), hb[g][3]);
    }
  }
  for (int j = TB; j < T; ++j) {
    const float xj = xs[j];
#pragma unroll
    for (int g = 0; g < OWN; ++g) {
      const u32x2_t q = in_weight(j, g);
      hb[g][0] = fmaf(xj, bf_lo(q[0]), hb[g][0]);
      hb[g][1] = fmaf(xj, bf_hi(q[0]), hb[g][1]);
      hb[g][2] = fmaf(xj, bf_lo(q[1]), hb[g][2]);
      hb[g][3] = fmaf(xj, bf_hi(q[1]), hb[g][3]);
    }
  }
#pragma unroll
  for (int g = 0; g < OWN; ++g) bstore16(r_h, col[g] * 4, __builtin_bit_cast(u32x4_t, hb[g]));
  if (!a.m_next) return;
  // (every wave's reads of the row before lie ahead of the barriers above)
#pragma unroll
  for (int g = 0; g < OWN; ++g) row_v[p][wr + g * nwr][lane] = hb[g];
  __syncthreads();
  f32x4_t v[GT];
  gather(v);
  float mean, rstd;
  row_stats(v, in_row, w, a.eps_ln, mean, rstd);
  const rsrc_t r_u = make_out(a.u + row * w, row2);
#pragma unroll
  for (int g = 0; g < OWN; ++g) {
    mod4(hb[g], mean, rstd, sh2[g], sc2[g]);
    __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{pack2bf(hb[g][0], hb[g][1]), pack2bf(hb[g][2], hb[g][3])}, r_u, col[g] * 2,
                                          0, 0);
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Handle and C ABI
// ---------------------------------------------------------------------------

// Scratch of one call: 2R rows of the network's activations (R tokens) and
// the R latents; s and m hold the rows of `steps` sampling steps.
struct HeadScratch {
  bf16_t* a0;  // [2R, cond_dim]
  float* c;    // [2R, w]
  bf16_t* s;   // [steps 2R, w]
  bf16_t* m;   // [steps 2R, n_mod w]
  float* h;    // [2R, w]
  bf16_t* u;   // [2R, w]
  bf16_t* g;   // [2R, w]
  float* x;    // [R, T]
};

struct mar_head {
  mar_head_dims d;
  int n_mod;
  // weights (matrices bf16, biases fp32)
  void *z_w, *t1_w, *t2_w, *in_w, *ada_w, *fc1_w, *fc2_w, *out_w;
  float *z_b, *t1_b, *t2_b, *in_b, *ada_b, *fc1_b, *fc2_b, *out_b;
  bf16_t* in_wt;   // [T, w] the input product's weights, transposed
  float* e;        // [steps, w] time embeddings
  f32x4_t* coef;   // [steps] DDPM coefficients
  bf16_t* phi;     // [steps, freq] (init only)
  bf16_t* t1o;     // [steps, w] (init only)
  HeadScratch sc;  // in the workspace, for up to max_rows tokens
  size_t mod_rows; // rows that its s and m hold
};

namespace {

mar_status check_head_dims(const mar_head_dims* d) {
  if (!d) return hfail(MAR_E_ARG, "dims is NULL");
  if (d->dtype != MAR_BF16) return hfail(MAR_E_ARG, "the diffusion head runs in bf16 (dtype %d)", d->dtype);
  if (d->width < 64 || d->width % 64 || d->width > 4096)
    return hfail(MAR_E_SHAPE, "width %d must be a multiple of 64 in [64, 4096]", d->width);
  if (d->depth < 1) return hfail(MAR_E_SHAPE, "depth must be >= 1");
  if (d->cond_dim < 64 || d->cond_dim % 64 || d->cond_dim > 4096)
    return hfail(MAR_E_SHAPE, "cond_dim %d must be a multiple of 64 in [64, 4096]", d->cond_dim);
  if (d->token_dim < 1 || d->token_dim > 64) return hfail(MAR_E_SHAPE, "token_dim must be in [1, 64]");
  if (d->freq_dim < 64 || d->freq_dim % 64 || d->freq_dim > 1024)
    return hfail(MAR_E_SHAPE, "freq_dim must be a multiple of 64 in [64, 1024]");
  if (d->steps < 1 || d->train_steps < d->steps || d->train_steps > 100000)
    return hfail(MAR_E_SHAPE, "need 1 <= steps <= train_steps <= 100000");
  if (!(d->beta_start > 0.f) || !(d->beta_end >= d->beta_start) || !(d->beta_end < 1.f))
    return hfail(MAR_E_ARG, "need 0 < beta_start <= beta_end < 1");
  if (!(d->ln_eps > 0.f)) return hfail(MAR_E_ARG, "ln_eps must be positive");
  if (d->max_rows < 1 || d->max_rows > 65536) return hfail(MAR_E_SHAPE, "max_rows must be in [1, 65536]");
  const size_t n_mod = 3 * static_cast<size_t>(d->depth) + 2;
  if (2 * static_cast<size_t>(d->max_rows) * n_mod * d->width * 4 >= (size_t(1) << 31))
    return hfail(MAR_E_SHAPE, "2 max_rows (3 depth + 2) width * 4 reaches 2 GiB (32-bit offsets)");
  return MAR_OK;
}

// Sampling steps whose modulation rows are made in one product, for calls of
// `rows` tokens: 2048 rows' worth.  The product of one step (512 x 33280 x
// 1280 at 256 tokens, four rounds of half-size tiles on two workgroups per CU)
// took 50 us on MI355X; four steps' 170 us (42 a step), eight steps' 320 us,
// which is not worth the scratch (136 MB for four at width 1280, 8 blocks).
// At 5 tokens of width 1024 it was 11.7 us a step for 10 rows.
constexpr size_t kModRows = 2048;
size_t most_mod_rows(const mar_head_dims& d) {  // 32-bit offsets of the product, as for one step
  return std::min(kModRows, ((size_t(1) << 31) - 1) / ((3 * static_cast<size_t>(d.depth) + 2) * d.width * 4));
}
size_t mod_steps(const mar_head_dims& d, size_t rows) {
  return std::max<size_t>(1, std::min<size_t>(most_mod_rows(d) / (2 * rows), d.steps));
}

// Byte offsets of the scratch of a call on `rows` tokens with the modulation
// rows of `steps` sampling steps (256-byte aligned, from 0, in the order of
// HeadScratch's fields); returns its size.
constexpr int kScratchBuffers = 8;
size_t scratch_layout(const mar_head_dims& d, size_t rows, size_t mod_rows, size_t* off) {
  const size_t w = d.width, D = d.cond_dim, T = d.token_dim;
  const size_t nm = 3 * static_cast<size_t>(d.depth) + 2, R2 = 2 * rows;
  const size_t sizes[kScratchBuffers] = {R2 * D * 2, R2 * w * 4, mod_rows * w * 2, mod_rows * nm * w * 2,
                                         R2 * w * 4, R2 * w * 2, R2 * w * 2, rows * T * 4};
  size_t o = 0;
  for (int k = 0; k < kScratchBuffers; ++k) {
    off[k] = o;
    o = align_up(o + sizes[k]);
  }
  return o;
}

// Modulation rows that a workspace of mar_head_workspace_bytes() holds: one
// step's of max_rows tokens, or kModSteps steps' as far as mod_steps() can ask
// for them.  All 100 steps of a small handle at once gain nothing over 16 and
// take six times the memory: 5 tokens, 7 at most, of the width 1280 head took
// 8163 us on MI355X with 100 steps' rows (97 MB), 8221 with 16 (16 MB), 8327
// with 8, 10074 with one (1.2 MB); of the width 1024 head 5608, 5651, 5738,
// 6885 us.
constexpr size_t kModSteps = 16;
size_t workspace_mod_rows(const mar_head_dims& d) {
  const size_t all = 2 * static_cast<size_t>(d.max_rows);
  return std::max(all, std::min(all * std::min<size_t>(d.steps, kModSteps), most_mod_rows(d)));
}

HeadScratch scratch_at(unsigned char* base, const size_t* off) {
  HeadScratch sc;
  sc.a0 = reinterpret_cast<bf16_t*>(base + off[0]);
  sc.c = reinterpret_cast<float*>(base + off[1]);
  sc.s = reinterpret_cast<bf16_t*>(base + off[2]);
  sc.m = reinterpret_cast<bf16_t*>(base + off[3]);
  sc.h = reinterpret_cast<float*>(base + off[4]);
  sc.u = reinterpret_cast<bf16_t*>(base + off[5]);
  sc.g = reinterpret_cast<bf16_t*>(base + off[6]);
  sc.x = reinterpret_cast<float*>(base + off[7]);
  return sc;
}

// Byte offsets of the weights and tables in the workspace (in the order of
// mar_head's fields), followed by the scratch for max_rows tokens at
// off[kTables]; returns the total.
constexpr int kTables = 21;
size_t head_layout(const mar_head_dims& d, size_t* off) {
  const size_t w = d.width, D = d.cond_dim, T = d.token_dim, F = d.freq_dim, S = d.steps;
  const size_t nm = 3 * static_cast<size_t>(d.depth) + 2, L = d.depth;
  const size_t sizes[kTables] = {
      w * D * 2, w * F * 2, w * w * 2, w * T * 2, nm * w * w * 2, L * w * w * 2, L * w * w * 2, T * w * 2,
      w * 4, w * 4, w * 4, w * 4, nm * w * 4, L * w * 4, L * w * 4, T * 4,
      S * w * 4, S * 16, S * F * 2, S * w * 2, T * w * 2};
  size_t o = 0;
  for (int k = 0; k < kTables; ++k) {
    off[k] = o;
    o = align_up(o + sizes[k]);
  }
  off[kTables] = o;
  size_t soff[kScratchBuffers];
  return o + scratch_layout(d, static_cast<size_t>(d.max_rows), workspace_mod_rows(d), soff);
}
constexpr int kHeadBuffers = kTables + 1;

template <class Kern, class... Args>
hipError_t launch_rows(Kern k, int rows, hipStream_t st, Args... args) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k, dim3((rows + 3) / 4), dim3(256), 0, st, args...);
  return hipGetLastError();
}

// ln-modulation and output kernels by the groups of 4 a lane holds
template <int G, bool EXACT>
hipError_t lnmod_as(const mar_head* hd, const HeadScratch& sc, const bf16_t* m, int off_shift, int off_scale, int rows,
                    hipStream_t st) {
  return launch_rows(head_lnmod_kernel<G, EXACT>, rows, st, static_cast<const float*>(sc.h),
                     m, hd->n_mod * hd->d.width, off_shift, off_scale, rows, hd->d.width, hd->d.ln_eps, sc.u);
}
hipError_t launch_lnmod(const mar_head* hd, const HeadScratch& sc, const bf16_t* m, int off_shift, int off_scale, int rows,
                        hipStream_t st) {
  switch (hd->d.width) {
    case 1024: return lnmod_as<4, true>(hd, sc, m, off_shift, off_scale, rows, st);
    case 1280: return lnmod_as<5, true>(hd, sc, m, off_shift, off_scale, rows, st);
    case 1536: return lnmod_as<6, true>(hd, sc, m, off_shift, off_scale, rows, st);
    default: break;
  }
  const int G = (hd->d.width + 255) / 256;
  if (G <= 2) return lnmod_as<2, false>(hd, sc, m, off_shift, off_scale, rows, st);
  if (G <= 4) return lnmod_as<4, false>(hd, sc, m, off_shift, off_scale, rows, st);
  if (G <= 8) return lnmod_as<8, false>(hd, sc, m, off_shift, off_scale, rows, st);
  return lnmod_as<16, false>(hd, sc, m, off_shift, off_scale, rows, st);
}
// The step kernel: a wave per 256 columns up to width 2048, per 512 beyond,
// and the output components over as many of a row's waves as there are (16, 8,
// 4 or 2 each: powers of two, for the halving exchanges).
hipError_t launch_step(const mar_head* hd, StepArgs a, hipStream_t st) {
  const int groups = (a.w + 255) / 256;
  a.nwr = groups <= 8 ? groups : (groups + 1) / 2;
  auto kern = head_step_kernel<16, 4>;
  switch (groups) {
    case 1: kern = head_step_kernel<1, 16>; break;
    case 2: kern = head_step_kernel<2, 8>; break;
    case 3: kern = head_step_kernel<3, 8>; break;
    case 4: kern = head_step_kernel<4, 4>; break;
    case 5: kern = head_step_kernel<5, 4>; break;
    case 6: kern = head_step_kernel<6, 4>; break;
    case 7: kern = head_step_kernel<7, 4>; break;
    case 8: kern = head_step_kernel<8, 2>; break;
    default: break;
  }
  hipLaunchKernelGGL(kern, dim3(a.R), dim3(128 * a.nwr), 0, st, a);
  return hipGetLastError();
}

hipError_t fill_zero(float* p, long n, hipStream_t st) {
  const long n4 = n / 4;  // every zeroed buffer holds a multiple of 4 floats
  if (n4 <= 0) return hipSuccess;
  hipLaunchKernelGGL(head_fill_zero_kernel, dim3((n4 + 255) / 256), dim3(256), 0, st, p, n4);
  return hipGetLastError();
}

hipError_t gemm(const void* a, const void* w, int M, int N, int K, const EpiArgs& e, hipStream_t st) {
  return launch_gemm(DT_BF16, a, w, M, N, K, e, st);
}

mar_status head_init(const mar_head_dims* dims, const mar_head_weights* W, void* workspace, size_t bytes,
                     void* stream, mar_head** out) {
  if (!out) return hfail(MAR_E_ARG, "out is NULL");
  *out = nullptr;
  mar_status s = check_head_dims(dims);
  if (s != MAR_OK) return s;
  if (!W) return hfail(MAR_E_ARG, "weights is NULL");
  const void* ptrs[] = {W->z_w, W->z_b, W->t1_w, W->t1_b, W->t2_w, W->t2_b, W->in_w, W->in_b,
                        W->ada_w, W->ada_b, W->fc1_w, W->fc1_b, W->fc2_w, W->fc2_b, W->out_w, W->out_b};
  for (const void* p : ptrs)
    if (!p) return hfail(MAR_E_ARG, "a weight pointer is NULL");
  if (!workspace) return hfail(MAR_E_ARG, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign) return hfail(MAR_E_WORKSPACE, "workspace must be 256-byte aligned");
  const mar_head_dims& d = *dims;
  size_t off[kHeadBuffers], soff[kScratchBuffers];
  head_layout(d, off);
  // the modulation rows of one sampling step have to fit; of more, as many as do
  size_t mod_rows = 2 * static_cast<size_t>(d.max_rows), most = workspace_mod_rows(d);
  auto need = [&](size_t rows) { return off[kTables] + scratch_layout(d, static_cast<size_t>(d.max_rows), rows, soff); };
  if (bytes < need(mod_rows))
    return hfail(MAR_E_WORKSPACE, "workspace holds %zu bytes, %zu needed", bytes, need(mod_rows));
  while (mod_rows < most) {
    const size_t mid = (mod_rows + most + 1) / 2;
    if (need(mid) <= bytes) mod_rows = mid;
    else most = mid - 1;
  }
  std::unique_ptr<mar_head> hd(new (std::nothrow) mar_head);
  if (!hd) return hfail(MAR_E_HOST, "out of host memory");
  hd->d = d;
  hd->n_mod = 3 * d.depth + 2;
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  void** mats[] = {&hd->z_w, &hd->t1_w, &hd->t2_w, &hd->in_w, &hd->ada_w, &hd->fc1_w, &hd->fc2_w, &hd->out_w};
  float** vecs[] = {&hd->z_b, &hd->t1_b, &hd->t2_b, &hd->in_b, &hd->ada_b, &hd->fc1_b, &hd->fc2_b, &hd->out_b};
  for (int k = 0; k < 8; ++k) *mats[k] = ws + off[k];
  for (int k = 0; k < 8; ++k) *vecs[k] = reinterpret_cast<float*>(ws + off[8 + k]);
  hd->e = reinterpret_cast<float*>(ws + off[16]);
  hd->coef = reinterpret_cast<f32x4_t*>(ws + off[17]);
  hd->phi = reinterpret_cast<bf16_t*>(ws + off[18]);
  hd->t1o = reinterpret_cast<bf16_t*>(ws + off[19]);
  hd->in_wt = reinterpret_cast<bf16_t*>(ws + off[20]);
  hd->mod_rows = mod_rows;
  scratch_layout(d, static_cast<size_t>(d.max_rows), hd->mod_rows, soff);
  hd->sc = scratch_at(ws + off[kTables], soff);

  hipStream_t st = static_cast<hipStream_t>(stream);
  const size_t w = d.width, D = d.cond_dim, T = d.token_dim, F = d.freq_dim, L = d.depth, nm = hd->n_mod;
  struct Cp { void* dst; const void* src; size_t bytes; } cps[] = {
      {hd->z_w, W->z_w, w * D * 2},       {hd->t1_w, W->t1_w, w * F * 2},    {hd->t2_w, W->t2_w, w * w * 2},
      {hd->in_w, W->in_w, w * T * 2},     {hd->ada_w, W->ada_w, nm * w * w * 2},
      {hd->fc1_w, W->fc1_w, L * w * w * 2}, {hd->fc2_w, W->fc2_w, L * w * w * 2}, {hd->out_w, W->out_w, T * w * 2},
      {hd->z_b, W->z_b, w * 4},           {hd->t1_b, W->t1_b, w * 4},        {hd->t2_b, W->t2_b, w * 4},
      {hd->in_b, W->in_b, w * 4},         {hd->ada_b, W->ada_b, nm * w * 4}, {hd->fc1_b, W->fc1_b, L * w * 4},
      {hd->fc2_b, W->fc2_b, L * w * 4},   {hd->out_b, W->out_b, T * 4}};
  for (const Cp& cp : cps) HEAD_HIP(hipMemcpyAsync(cp.dst, cp.src, cp.bytes, hipMemcpyDeviceToDevice, st), "weight copy");
  // the sampler's coefficients and the time embedding of every step
  hipLaunchKernelGGL(head_schedule_kernel, dim3(1), dim3(64), 0, st, d.steps, d.train_steps,
                     static_cast<double>(d.beta_start), static_cast<double>(d.beta_end), hd->coef);
  HEAD_HIP(hipGetLastError(), "schedule");
  hipLaunchKernelGGL(head_phi_kernel, dim3(d.steps), dim3(256), 0, st, static_cast<const f32x4_t*>(hd->coef), d.steps,
                     d.freq_dim, hd->phi);
  HEAD_HIP(hipGetLastError(), "time features");
  EpiArgs e1{};
  e1.kind = EPI_SILU;
  e1.bias = hd->t1_b;
  e1.out = hd->t1o;
  HEAD_HIP(gemm(hd->phi, hd->t1_w, d.steps, d.width, d.freq_dim, e1, st), "time embedding (first product)");
  HEAD_HIP(fill_zero(hd->e, static_cast<long>(d.steps) * d.width, st), "zero fill");
  EpiArgs e2{};
  e2.kind = EPI_RESIDUAL;
  e2.bias = hd->t2_b;
  e2.out = hd->e;
  e2.resid = hd->e;
  HEAD_HIP(gemm(hd->t1o, hd->t2_w, d.steps, d.width, d.width, e2, st), "time embedding (second product)");
  {
    const long n = static_cast<long>(d.width) * d.token_dim;
    hipLaunchKernelGGL(head_transpose_in_kernel, dim3((n + 255) / 256), dim3(256), 0, st,
                       static_cast<const bf16_t*>(hd->in_w), d.width, d.token_dim, hd->in_wt);
    HEAD_HIP(hipGetLastError(), "input weights");
  }
  *out = hd.release();
  return MAR_OK;
}

// Arguments of a call, checked on the host (rows against the caller's
// limit, which the scratch behind the call must hold).
mar_status check_sample(const mar_head* hd, const float* yc, const float* yu, int32_t y_rows, const int32_t* rc,
                        const int32_t* ru, int32_t R, int32_t max_R, const float* x_init, const float* xi,
                        float scale, float* x_out, float* traj, float* eps_out) {
  if (!hd) return hfail(MAR_E_ARG, "head is NULL");
  if (R < 0 || R > max_R) return hfail(MAR_E_ARG, "rows %d outside [0, %d]", R, max_R);
  if (R == 0) return MAR_OK;
  if (!yc || !yu || !rc || !ru || !x_init || !xi || !x_out) return hfail(MAR_E_ARG, "NULL pointer");
  if (y_rows < 1) return hfail(MAR_E_ARG, "y_rows must be >= 1");
  const void* al[] = {yc, yu, x_init, xi, x_out, traj ? traj : x_out, eps_out ? eps_out : x_out};
  for (const void* p : al)
    if (!aligned16(p)) return hfail(MAR_E_ARG, "float buffers must be 16-byte aligned");
  if (!std::isfinite(scale)) return hfail(MAR_E_ARG, "scale must be finite");
  {
    hipError_t e = hipPeekAtLastError();
    if (e != hipSuccess) return hfail(MAR_E_DEVICE, "earlier device error: %s", hipGetErrorString(e));
  }
  return MAR_OK;
}

// The sampler over R >= 1 tokens with the scratch `sc`, whose s and m hold
// mod_rows >= 2R rows (checked arguments).
mar_status head_sample(const mar_head* hd, const HeadScratch& sc, size_t mod_rows, const float* yc, const float* yu, int32_t y_rows,
                       const int32_t* rc, const int32_t* ru, int32_t R, const float* x_init, const float* xi,
                       float scale, float* x_out, float* traj, float* eps_out, void* stream) {
  const mar_head_dims& d = hd->d;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int w = d.width, D = d.cond_dim, T = d.token_dim, R2 = 2 * R, nm = hd->n_mod;
  const size_t xbytes = static_cast<size_t>(R) * T * sizeof(float);
  HEAD_HIP(launch_rows(head_gather_kernel, R2, st, yc, yu, static_cast<int>(y_rows), rc, ru, static_cast<int>(R), D,
                       sc.a0),
           "gather");
  HEAD_HIP(fill_zero(sc.c, static_cast<long>(R2) * w, st), "zero fill");
  EpiArgs ec{};
  ec.kind = EPI_RESIDUAL;
  ec.bias = hd->z_b;
  ec.out = sc.c;
  ec.resid = sc.c;
  HEAD_HIP(gemm(sc.a0, hd->z_w, R2, w, D, ec, st), "conditioning product");
  HEAD_HIP(hipMemcpyAsync(sc.x, x_init, xbytes, hipMemcpyDeviceToDevice, st), "latent copy");
  if (traj) HEAD_HIP(hipMemcpyAsync(traj, x_init, xbytes, hipMemcpyDeviceToDevice, st), "trajectory copy");
  StepArgs sa{};
  sa.out_w = static_cast<const bf16_t*>(hd->out_w);
  sa.in_wt = hd->in_wt;
  sa.out_b = hd->out_b;
  sa.in_b = hd->in_b;
  sa.xi = xi;
  sa.coef = hd->coef;
  sa.h = sc.h;
  sa.x = sc.x;
  sa.u = sc.u;
  sa.ld = nm * w;
  sa.shift_out = 3 * d.depth * w;
  sa.scale_out = (3 * d.depth + 1) * w;
  sa.R = R;
  sa.w = w;
  sa.T = T;
  sa.eps_ln = d.ln_eps;
  sa.scale = scale;
  const int batch = static_cast<int>(std::min(mod_steps(d, R), mod_rows / R2));
  for (int j = 0; j < d.steps; ++j) {
    const int i = d.steps - 1 - j;
    const int at = j % batch;  // this step's place among the steps whose modulation was made together
    bf16_t* m = sc.m + static_cast<long>(at) * R2 * nm * w;
    if (at == 0) {
      const int C = std::min(batch, d.steps - j);
      HEAD_HIP(launch_rows(head_silu_kernel, C * R2, st, static_cast<const float*>(sc.c),
                           static_cast<const float*>(hd->e), i, C, R2, w, sc.s),
               "conditioning");
      EpiArgs em{};
      em.kind = EPI_BIAS;
      em.bias = hd->ada_b;
      em.out = sc.m;
      HEAD_HIP(gemm(sc.s, hd->ada_w, C * R2, nm * w, w, em, st), "modulation product");
      if (j == 0) {
        StepArgs first = sa;
        first.next = 1;
        first.m_next = m;
        HEAD_HIP(launch_step(hd, first, st), "input product");
      } else {
        HEAD_HIP(launch_lnmod(hd, sc, m, 0, w, R2, st), "ln-modulation");
      }
    }
    for (int k = 0; k < d.depth; ++k) {
      if (k > 0) HEAD_HIP(launch_lnmod(hd, sc, m, 3 * k * w, (3 * k + 1) * w, R2, st), "ln-modulation");
      EpiArgs e1{};
      e1.kind = EPI_SILU;
      e1.bias = hd->fc1_b + static_cast<long>(k) * w;
      e1.out = sc.g;
      HEAD_HIP(gemm(sc.u, static_cast<const bf16_t*>(hd->fc1_w) + static_cast<long>(k) * w * w, R2, w, w, e1, st),
               "block first product");
      EpiArgs e2{};
      e2.kind = EPI_GATE;
      e2.bias = hd->fc2_b + static_cast<long>(k) * w;
      e2.out = sc.h;
      e2.resid = sc.h;
      e2.gate = m + static_cast<long>(3 * k + 2) * w;
      e2.gate_ld = nm * w;
      HEAD_HIP(gemm(sc.g, static_cast<const bf16_t*>(hd->fc2_w) + static_cast<long>(k) * w * w, R2, w, w, e2, st),
               "block second product");
    }
    StepArgs step = sa;
    step.out = 1;
    step.next = j + 1 < d.steps;
    step.m_out = m;
    step.m_next = step.next && at + 1 < batch ? m + static_cast<long>(R2) * nm * w : nullptr;
    step.i = i;
    step.traj = traj ? traj + static_cast<long>(j + 1) * R * T : nullptr;
    step.eps_out = eps_out ? eps_out + static_cast<long>(j) * R * T : nullptr;
    HEAD_HIP(launch_step(hd, step, st), "output and sampler step");
  }
  HEAD_HIP(hipMemcpyAsync(x_out, sc.x, xbytes, hipMemcpyDeviceToDevice, st), "latent copy");
  return MAR_OK;
}

// ---------------------------------------------------------------------------
// Scratch of mar_head_sample_noalloc: one file-scope array per GPU, for
// callers that cannot allocate device memory.  In host code `scratch` names
// a host-side stand-in; the array's device address comes from
// hipGetSymbolAddress, resolved once per device (at init, else at the
// first call on that device) and kept in kScratchPtr.
// ---------------------------------------------------------------------------
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array.
mar_status static_scratch(void** out) {
  int dev = -1;
  HEAD_HIP(hipGetDevice(&dev), "current device");
  if (dev < 0 || dev >= kMaxDevices) return hfail(MAR_E_DEVICE, "device %d beyond the scratch table", dev);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HEAD_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "scratch address");
    if (!p) return hfail(MAR_E_DEVICE, "scratch address is NULL");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return MAR_OK;
}

}  // namespace

extern "C" {

size_t mar_head_workspace_bytes(const mar_head_dims* dims) {
  abi_clear_error();
  if (check_head_dims(dims) != MAR_OK) return 0;
  size_t off[kHeadBuffers];
  return head_layout(*dims, off);
}

mar_status mar_head_init(const mar_head_dims* dims, const mar_head_weights* weights, void* workspace,
                         size_t workspace_bytes, void* stream, mar_head** out) {
  abi_clear_error();
  try {
    mar_status s = head_init(dims, weights, workspace, workspace_bytes, stream, out);
    if (s != MAR_OK) return s;
    void* p = nullptr;
    s = static_scratch(&p);  // the allocation-free entry point's array, resolved here once per device
    if (s != MAR_OK) {
      delete *out;
      *out = nullptr;
    }
    return s;
  } catch (const std::bad_alloc&) {
    return hfail(MAR_E_HOST, "out of host memory");
  } catch (const std::system_error&) {
    return hfail(MAR_E_HOST, "lock failed");
  }
}

mar_status mar_head_sample(mar_head* head, const float* y_cond, const float* y_uncond, int32_t y_rows,
                           const int32_t* row_cond, const int32_t* row_uncond, int32_t rows, const float* x_init,
                           const float* xi, float scale, float* x_out, float* trajectory, float* eps_out,
                           void* stream) {
  abi_clear_error();
  mar_status s = check_sample(head, y_cond, y_uncond, y_rows, row_cond, row_uncond, rows,
                              head ? head->d.max_rows : 0, x_init, xi, scale, x_out, trajectory, eps_out);
  if (s != MAR_OK || rows == 0) return s;
  return head_sample(head, head->sc, head->mod_rows, y_cond, y_uncond, y_rows, row_cond, row_uncond, rows, x_init, xi, scale, x_out,
                     trajectory, eps_out, stream);
}

mar_status mar_head_sample_noalloc(mar_head* head, const float* y_cond, const float* y_uncond, int32_t y_rows,
                                   const int32_t* row_cond, const int32_t* row_uncond, int32_t rows,
                                   const float* x_init, const float* xi, float scale, float* x_out,
                                   float* trajectory, float* eps_out, void* stream) {
  abi_clear_error();
  mar_status s = check_sample(head, y_cond, y_uncond, y_rows, row_cond, row_uncond, rows, 65536, x_init, xi, scale,
                              x_out, trajectory, eps_out);
  if (s != MAR_OK || rows == 0) return s;
  // the modulation rows of as many steps as mod_steps() asks for and the
  // array holds next to the rest
  size_t off[kScratchBuffers];
  const size_t R2 = 2 * static_cast<size_t>(rows);
  size_t steps = mod_steps(head->d, rows);
  while (steps > 1 && scratch_layout(head->d, rows, steps * R2, off) > kStaticScratchBytes) --steps;
  const size_t need = scratch_layout(head->d, rows, steps * R2, off);
  if (need > kStaticScratchBytes)
    return hfail(MAR_E_SHAPE, "%d rows need %zu bytes of scratch; the static array holds %zu", rows, need,
                 kStaticScratchBytes);
  void* base = nullptr;
  try {
    s = static_scratch(&base);
  } catch (const std::system_error&) {
    return hfail(MAR_E_HOST, "lock failed");
  }
  if (s != MAR_OK) return s;
  return head_sample(head, scratch_at(static_cast<unsigned char*>(base), off), steps * R2, y_cond, y_uncond, y_rows, row_cond,
                     row_uncond, rows, x_init, xi, scale, x_out, trajectory, eps_out, stream);
}

mar_status mar_head_destroy(mar_head* head) {
  delete head;
  return MAR_OK;
}

}  // extern "C"
