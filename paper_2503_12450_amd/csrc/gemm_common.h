// What the product kernels share: the epilogues' activations (the same
// functions everywhere, so the choice of kernel never changes a result bit),
// the loads into LDS and their waits, and the map from workgroups to output
// tiles.
#pragma once

#include "common.h"

namespace marcache {

// GELU x * Phi(x) = 0.5 x (1 + erf(x / sqrt 2)), with erf from Abramowitz &
// Stegun, Handbook of Mathematical Functions, formula 7.1.26:
//   erf(z) = 1 - (a1 t + a2 t^2 + a3 t^3 + a4 t^4 + a5 t^5) exp(-z^2),
//   t = 1 / (1 + p z), z >= 0, |error| <= 1.5e-7,
// far below the bf16 rounding of the product it feeds.  With
// q = (1 - erf(|x| / sqrt 2)) / 2:  gelu(x) = x (1 - q) for x >= 0, x q else.
__device__ __forceinline__ float gelu_erf(float x) {
  const float z = fabsf(x) * 0.70710678118654752440f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
  float poly = fmaf(1.061405429f, t, -1.453152027f);
  poly = fmaf(poly, t, 1.421413741f);
  poly = fmaf(poly, t, -0.284496736f);
  poly = fmaf(poly, t, 0.254829592f);
  poly *= t;
  const float q = 0.5f * poly * __expf(-z * z);
  return x >= 0.0f ? x * (1.0f - q) : x * q;
}

// The same GELU for outputs stored in bf16, with erf from Abramowitz &
// Stegun formula 7.1.27:
//   erf(z) = 1 - 1 / (1 + a1 z + a2 z^2 + a3 z^3 + a4 z^4)^4,  z >= 0,
//   |error| <= 5e-4,
// so with z = |x| / sqrt(2), q = (1 - erf(z)) / 2 = 1 / (2^(1/4) D)^4: the
// polynomial is taken in |x| with its coefficients scaled by 2^(1/4) and
// powers of 1/sqrt(2), and one reciprocal gives q.  gelu = x (1 - q) for
// x >= 0 and x q for x < 0, which is max(x, 0) - |x| q for both signs.
// The error in gelu is at most 2.4e-4 |x|: a sixteenth of the bf16 step of x,
// and so of the result for x > 0.  In the negative tail, where the result is
// far smaller than x, that is an absolute bound only: relative to the result
// it is 0.8 % at x = -2, 17 % at -3 and more than the result from -4 on.
__device__ __forceinline__ float gelu_erf_bf16(float x) {
  const float ax = fabsf(x);
  float d = fmaf(0.0232216473f, ax, 0.000408675658f);  // 2^(1/4) (a4 / 4, a3 / 2^(3/2))
  d = fmaf(d, ax, 0.136990119f);                       // 2^(1/4) a2 / 2
  d = fmaf(d, ax, 0.234099676f);                       // 2^(1/4) a1 / 2^(1/2)
  d = fmaf(d, ax, 1.18920712f);                        // 2^(1/4)
  const float r = __builtin_amdgcn_rcpf(d);
  const float r2 = r * r;
  return fmaf(-(ax * r2), r2, fmaxf(x, 0.0f));
}

// silu(x) = x / (1 + e^-x), with the hardware exp2 and reciprocal (each
// within a few fp32 ulps; the result is stored in bf16).  For x below
// about -88 the exponential overflows to +inf and the quotient is -0,
// the limit.
__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

typedef __attribute__((ext_vector_type(4))) int i32x4_t;

// Buffer descriptor over `bytes` bytes at `base` (raw, no stride).
__device__ __forceinline__ i32x4_t make_rsrc(const void* base, unsigned bytes) {
  const unsigned long p = reinterpret_cast<unsigned long>(base);
  i32x4_t r;
  r[0] = __builtin_amdgcn_readfirstlane(static_cast<int>(p & 0xFFFFFFFFu));
  r[1] = __builtin_amdgcn_readfirstlane(static_cast<int>(p >> 32));
  r[2] = __builtin_amdgcn_readfirstlane(static_cast<int>(bytes));
  r[3] = 0x00020000;
  return r;
}

// Sixteen bytes per lane from the buffer (byte offset voff + soff) into LDS at
// lds_addr + 16 * lane.  Issued from asm so the compiler adds no waits of its
// own (it would drain every load before each LDS read); the main loop waits
// with s_waitcnt vmcnt for exactly the slice it is about to read.
// m0 is reserved by the compiler but nothing else in these kernels uses it
// (no LDS-DMA builtins, GWS or messages), so clobbering it here is safe.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(i32x4_t rsrc, unsigned lds_addr, int voff, int soff) {
  // the descriptor is wave-uniform; readfirstlane keeps it in SGPRs even
  // when it was picked by a select (a no-op when it is scalar already)
  i32x4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_readfirstlane(rsrc[i]);
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(r), "s"(soff)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// Workgroup barrier that waits for this wave's LDS operations only (a
// __syncthreads would also drain the vector-memory counter, i.e. the loads
// already in flight for later slices).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr int cmin(int a, int b) { return a < b ? a : b; }

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding).
// A wave has at most 63 such operations outstanding (issue stalls at that
// count), so a wait for "all but the last N" with N >= 63 is a wait for all
// but the last 63.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

constexpr int kOob = 0x7FFFFFF0;  // an offset past every descriptor

typedef __amdgpu_buffer_rsrc_t rsrc_t;

__device__ __forceinline__ rsrc_t make_out(void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, static_cast<int>(bytes), 0x00020000);
}
__device__ __forceinline__ void bstore16(rsrc_t r, int voff, const u32x4_t& v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, 0);
}
__device__ __forceinline__ u32x4_t bload16(rsrc_t r, int voff) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0);
}
// QKV column section of global column ng: 0 query, 1 key, 2 value
__device__ __forceinline__ int qkv_section(const EpiArgs& e, int ng) {
  return ng >= 2 * e.d_model ? 2 : (ng >= e.d_model ? 1 : 0);
}

// Workgroup -> output tile.  Workgroups are dispatched round-robin over the
// eight XCDs (workgroup b runs on XCD b % 8), and each XCD has its own L2.
// Each XCD is given a contiguous range of the tile order, and that order
// walks kGroupM row tiles before moving to the next column tile, so the
// ~32 workgroups an XCD runs at once share 4 row tiles of A and 8 column
// tiles of W instead of touching every row tile of A.  The map is a
// bijection for any tile count.
constexpr int kXcds = 8;
constexpr int kGroupM = 4;
__device__ __forceinline__ void tile_of(int b, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n;
  const int q = total / kXcds, r = total - q * kXcds;
  const int x = b % kXcds, l = b / kXcds;
  const int t = x * q + min(x, r) + l;  // position in the tile order
  const int group = kGroupM * tiles_n;
  const int g = t / group, first_m = g * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int in = t - g * group;
  tm = first_m + in % gm;
  tn = in / gm;
}

}  // namespace marcache
