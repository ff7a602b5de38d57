// Token scoring and selection (Sec. 3.2, Eq. 8).
//
// score: S(x_i) = <v_i, r_i> / (||v_i|| ||r_i||) between this step's value
//   row v_i and the previous step's r_i.  The D = H * dh elements of a row are
//   spread over the heads of the [slot, head, token, dh] cache layout, each
//   lane reads 16-byte chunks.  The products of
//   stored bf16/fp32 values are exact in fp64; each lane keeps an unevaluated
//   sum hi + lo of them (Knuth's two-sum moves every rounding error of hi
//   into lo), the wave combines the pairs the same way, and hi + lo is
//   rounded once.  The three dot products are therefore the exactly rounded
//   sums whatever the lane/summation order (unless the errors themselves
//   span more than 53 bits).  Zero norms give 1 (both rows zero) or 0.  The
//   wave then overwrites r_i with v_i, so the reference always holds the
//   last step's rows.
// select: per slot, the n tokens with the smallest score (NaN ranks as +inf,
//   ties to the lower index), written in ascending token order: the n
//   smallest in the strict total order (score, index).  The opposite rule (the
//   n largest scores: Table 3's strategy that caches the least similar tokens)
//   ranks by (-score, index), NaN again last.
#include <algorithm>

#include "common.h"

namespace marcache {

// Unevaluated fp64 sum hi + lo.
struct Sum2 {
  double hi, lo;
};

// hi + p = s + e exactly (two-sum, no assumption on magnitudes).
__device__ __forceinline__ void add2(Sum2& a, double p) {
  const double s = a.hi + p;
  const double bb = s - a.hi;
  const double e = (a.hi - (s - bb)) + (p - bb);
  a.hi = s;
  a.lo += e;
}

__device__ __forceinline__ double wave_sum2(Sum2 a) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double oh = __shfl_xor(a.hi, o, 64);
    const double ol = __shfl_xor(a.lo, o, 64);
    a.lo += ol;
    add2(a, oh);
  }
  return a.hi + a.lo;
}

// Whether the products of the 16 bf16 values in two vectors can be summed (per
// vector pair: 8 of them) in fp64 without rounding: all finite, and nonzero
// exponents within 16 of each other.  A product has 16 significant bits, so
// the sums then span at most 2 * 16 + 19 = 51 bits.
__device__ __forceinline__ bool exact_sums(const u32x4_t& a, const u32x4_t& r) {
  typedef __attribute__((ext_vector_type(2))) unsigned short u16x2_t;
  u16x2_t hi = {0, 0}, lo = {0xFFFF, 0xFFFF};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const u16x2_t m = __builtin_bit_cast(u16x2_t, (i < 4 ? a[i] : r[i - 4]) & 0x7FFF7FFFu);
    hi = __builtin_elementwise_max(hi, m);
    lo = __builtin_elementwise_min(lo, static_cast<u16x2_t>(m - u16x2_t{1, 1}));  // zeros wrap to the top
  }
  const int h = max(hi[0], hi[1]), l = min(lo[0], lo[1]);
  return h < 0x7F80 && h - l <= 16 * 128;
}

// One vector of the current row and of the reference into the three sums.
// The fp64 operations of the exact sums are what bounded the scores (three
// two-sums, 21 operations, per element: 62 us for 40960 rows of 1024 on
// MI355X, 33 us of memory).  For bf16 the eight products of a vector are first
// added plainly where that is exact, which it nearly always is, and one
// two-sum takes their sum.  Where it hardly ever is (exponents spread evenly
// over 32 binades), the check costs 4 to 7 % of the one-wave kernel (640 rows
// of 768: 4.2 -> 4.4 us).
struct RowSums {
  Sum2 dot{0.0, 0.0}, nv{0.0, 0.0}, nr{0.0, 0.0};
};
template <typename T>
__device__ __forceinline__ void add_vector(RowSums& s, const u32x4_t& vv, const u32x4_t& rr) {
  constexpr int PER = Elem<T>::kPer16B;
  float fv[PER], fr[PER];
  unpack16(vv, fv, static_cast<const T*>(nullptr));
  unpack16(rr, fr, static_cast<const T*>(nullptr));
  if constexpr (sizeof(T) == 2) {
    if (__builtin_amdgcn_ballot_w64(!exact_sums(vv, rr)) == 0) {
      double d = 0.0, n = 0.0, m = 0.0;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const double a = fv[i], r = fr[i];
        d = fma(a, r, d);
        n = fma(a, a, n);
        m = fma(r, r, m);
      }
      add2(s.dot, d);
      add2(s.nv, n);
      add2(s.nr, m);
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const double a = fv[i], r = fr[i];
    add2(s.dot, a * r);
    add2(s.nv, a * a);
    add2(s.nr, r * r);
  }
}

__device__ __forceinline__ double cosine(double vr, double vv, double rr) {
  const double den = sqrt(vv * rr);
  if (den == 0.0) return (vv == 0.0 && rr == 0.0) ? 1.0 : 0.0;
  return vr / den;
}

// One wave per token, its lanes over the whole row.
template <typename T>
__global__ __launch_bounds__(256) void scores_kernel(const T* __restrict__ v_cur, T* __restrict__ v_ref, int n_slots,
                                                     int H, int seq, int dh, uint32_t dh_magic, int dh_shift,
                                                     double* __restrict__ scores, int update_ref) {
  constexpr int PER = Elem<T>::kPer16B;
  const int lane = threadIdx.x & 63;
  const long token = static_cast<long>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (token >= static_cast<long>(n_slots) * seq) return;
  const int b = static_cast<int>(token / seq);
  const int t = static_cast<int>(token % seq);
  const int n_chunks = H * dh / PER;
  RowSums s;
  for (int c = lane; c < n_chunks; c += 64) {
    const int e = c * PER;
    const int h = div_by(e, dh_magic, dh_shift);
    const long off = ((static_cast<long>(b) * H + h) * seq + t) * dh + (e - h * dh);
    const u32x4_t vv = *reinterpret_cast<const u32x4_t*>(v_cur + off);
    const u32x4_t rr = *reinterpret_cast<const u32x4_t*>(v_ref + off);
    if (update_ref) *reinterpret_cast<u32x4_t*>(v_ref + off) = vv;
    add_vector<T>(s, vv, rr);
  }
  const double vr = wave_sum2(s.dot), vv = wave_sum2(s.nv), rr = wave_sum2(s.nr);
  if (lane == 0) scores[token] = cosine(vr, vv, rr);
}

// Many tokens: a wave takes 64 / CPR consecutive tokens of a slot, CPR =
// 16-byte chunks of a head's row (8 for 64 bf16 values), and walks the heads:
// its loads are one contiguous piece per head instead of one piece per head
// and token, and the sums meet in log2(CPR) exchanges instead of six.  40960
// rows of 16 x 64: 33 us (5.1 TB/s), 51 us with one wave per token on MI355X.
constexpr int kHeadsAhead = 4;
template <typename T>
__global__ __launch_bounds__(256) void scores_runs_kernel(const T* __restrict__ v_cur, T* __restrict__ v_ref,
                                                          int n_slots, int H, int seq, int dh,
                                                          double* __restrict__ scores, int update_ref) {
  constexpr int PER = Elem<T>::kPer16B;
  const int lane = threadIdx.x & 63;
  const int cpr = dh / PER, run = 64 / cpr;  // chunks per row, tokens per wave
  const int runs = (seq + run - 1) / run;    // per slot
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (w >= n_slots * runs) return;
  const int b = w / runs;
  const int tl = lane / cpr, c = lane - tl * cpr;
  const int t = (w - b * runs) * run + tl;
  const bool ok = tl < run && t < seq;
  const long stride = static_cast<long>(seq) * dh;  // between heads
  const long off = (static_cast<long>(b) * H * seq + (ok ? t : 0)) * dh + (ok ? c : 0) * PER;
  RowSums s;
  for (int h0 = 0; h0 < H; h0 += kHeadsAhead) {
    u32x4_t vv[kHeadsAhead], rr[kHeadsAhead];
#pragma unroll
    for (int i = 0; i < kHeadsAhead; ++i) {
      const bool in = ok && h0 + i < H;
      vv[i] = in ? *reinterpret_cast<const u32x4_t*>(v_cur + off + (h0 + i) * stride) : u32x4_t{0u, 0u, 0u, 0u};
      rr[i] = in ? *reinterpret_cast<const u32x4_t*>(v_ref + off + (h0 + i) * stride) : u32x4_t{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < kHeadsAhead; ++i) {
      if (update_ref && ok && h0 + i < H) *reinterpret_cast<u32x4_t*>(v_ref + off + (h0 + i) * stride) = vv[i];
      add_vector<T>(s, vv[i], rr[i]);
    }
  }
  // sum over the row's lanes, into its first; the pairs are exact, so the
  // order does not matter
  auto meet = [&](Sum2 a) {
    for (int o = 32; o > 0; o >>= 1) {
      if (o >= cpr) continue;
      const double oh = __shfl_down(a.hi, o, 64), ol = __shfl_down(a.lo, o, 64);
      if (c + o < cpr && c < o) {
        a.lo += ol;
        add2(a, oh);
      }
    }
    return a.hi + a.lo;
  };
  const double vr = meet(s.dot), vv = meet(s.nv), rr = meet(s.nr);
  if (ok && c == 0) scores[static_cast<long>(b) * seq + t] = cosine(vr, vv, rr);
}

// Exclusive sum of v over the workgroup's threads, and the total; `sums` is
// one int per wave, free for reuse after the caller's next barrier.
template <int THREADS>
__device__ __forceinline__ int block_scan(int v, int* sums, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(inc, o, 64);
    if (lane >= o) inc += u;
  }
  if (lane == 63) sums[wave] = inc;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    const int s = sums[w];
    before += w < wave ? s : 0;
    total += s;
  }
  return before + inc - v;
}

// A radix selection, one workgroup per slot, whose threads own PER consecutive
// tokens each as 64-bit keys in score order.  The key range's common
// leading bits are skipped; then each pass counts the candidates (the keys
// that still agree with the n-th smallest) by their next 8 bits and keeps the
// bin that holds it, until that bin is wanted whole or no bits are left (equal
// scores: lowest index first).  What bounds it is the latency of a pass (three
// barriers, about 0.7 us) and a launch; two or three passes are usual.
// Ranking every token against every other took 21 us at 320 tokens and 150 us
// at 1088 on MI355X.  A workgroup has no more waves than its slot fills:
// with 512 threads for every length 4096 slots of 16 tokens took 22 us and 1024
// of 32 8.3 us (ranked 12.4 and 5.5), now 5.3 and 4.1.
template <int THREADS, int PER>
__global__ __launch_bounds__(THREADS) void select_kernel(const double* __restrict__ scores, int seq, int n,
                                                                int largest, int32_t* __restrict__ idx) {
  typedef unsigned long long u64;
  __shared__ u64 lohi[2][THREADS / 64];
  __shared__ int hist[256];
  __shared__ int found[3];  // digit, candidates before it, candidates in it
  __shared__ int sums[2][THREADS / 64];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const double* s = scores + static_cast<long>(b) * seq;
  const int t0 = tid * PER;
  double raw[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) raw[i] = s[min(t0 + i, seq - 1)];  // past the end: the last one, never counted
  u64 key[PER];
  u64 lo_k = ~0ull, hi_k = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    double v = largest ? -raw[i] : raw[i];
    if (v != v) v = __builtin_huge_val();  // NaN ranks last
    v += 0.0;                              // -0 ties with +0
    const u64 u = __builtin_bit_cast(u64, v);
    key[i] = u ^ ((u >> 63) ? ~0ull : 1ull << 63);
    lo_k = min(lo_k, key[i]);
    hi_k = max(hi_k, key[i]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo_k = min(lo_k, static_cast<u64>(__shfl_xor(lo_k, o, 64)));
    hi_k = max(hi_k, static_cast<u64>(__shfl_xor(hi_k, o, 64)));
  }
  if (lane == 0) {
    lohi[0][tid >> 6] = lo_k;
    lohi[1][tid >> 6] = hi_k;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    lo_k = min(lo_k, lohi[0][w]);
    hi_k = max(hi_k, lohi[1][w]);
  }
  // The selection's state is the same in every lane: held in scalar registers,
  // so that the pass loop is a uniform branch.  This is not only for speed: an
  // earlier form of this kernel (eight tokens per thread, the state left in
  // each lane's registers, so that the compiler made an exec-masked loop of
  // it) gave wrong rows now and then on MI355X, with lanes out of the loop
  // early.  Its source has the same barriers and the same uniform values, and
  // neither it nor its assembly shows a race or a hazard: the cause is not
  // known.  This form has not shown the fault over several hundred sequences
  // per launch at every number of tokens per thread.
  auto uniform64 = [](u64 v) {
    const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<int>(v));
    const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32));
    return static_cast<u64>(hi) << 32 | lo;
  };
  const u64 first = uniform64(lo_k), range = first ^ uniform64(hi_k);
  // Candidates: keys whose bits from `bit` up equal `prefix`; keys below that
  // prefix are chosen, `need` of the `cand` candidates remain to be.
  int bit = range ? 64 - __builtin_clzll(range) : 0;  // 0 when all keys are equal
  u64 prefix = bit < 64 ? first >> bit : 0;
  int need = n, cand = seq;
  auto above = [&](u64 k) { return bit < 64 ? k >> bit : u64(0); };
  while (bit > 0 && need < cand) {
    const int width = min(8, bit), next = bit - width;
    for (int i = tid; i < 256; i += THREADS) hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (t0 + i < seq && above(key[i]) == prefix)
        atomicAdd(&hist[static_cast<int>(key[i] >> next) & ((1 << width) - 1)], 1);
    __syncthreads();
    if (tid < 64) {
      int c[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[q] = hist[4 * lane + q];
        sum += c[q];
      }
      int inc = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(inc, o, 64);
        if (lane >= o) inc += u;
      }
      int before = inc - sum;
      if (before < need && need <= inc) {  // exactly one lane
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (before < need && need <= before + c[q]) {
            found[0] = 4 * lane + q;
            found[1] = before;
            found[2] = c[q];
          }
          before += c[q];
        }
      }
    }
    __syncthreads();
    prefix = (prefix << width) | static_cast<unsigned>(__builtin_amdgcn_readfirstlane(found[0]));
    need -= __builtin_amdgcn_readfirstlane(found[1]);
    cand = __builtin_amdgcn_readfirstlane(found[2]);
    bit = next;
  }
  // the candidates wanted are the first `need` in index order (all of them,
  // or equal scores)
  unsigned chosen = 0, ties = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const u64 a = above(key[i]);
    const bool own = t0 + i < seq;
    chosen |= (own && a < prefix ? 1u : 0u) << i;
    ties |= (own && a == prefix ? 1u : 0u) << i;
  }
  int total;
  int left = need - block_scan<THREADS>(__popc(ties), sums[0], total);
  for (; ties != 0 && left > 0; --left) {
    chosen |= ties & -ties;
    ties &= ties - 1;
  }
  int to = block_scan<THREADS>(__popc(chosen), sums[1], total);
  int32_t* out = idx + static_cast<long>(b) * n;
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if ((chosen >> i) & 1u) {
      if (to < n) out[to] = t0 + i;  // always true: exactly n are chosen
      ++to;
    }
}

hipError_t launch_scores(int dtype, const void* v_cur, void* v_ref, int n_slots, int H, int seq,
                         int dh, double* scores, bool update_ref, hipStream_t st) {
  const long tokens = static_cast<long>(n_slots) * seq;
  if (tokens == 0) return hipSuccess;
  const int cpr = dh / (dtype == DT_BF16 ? 8 : 4);
  if (H > 1 && cpr <= 32) {
    const int runs = (seq + 64 / cpr - 1) / (64 / cpr);
    // with fewer than four waves per CU one wave per token is faster: a run's
    // wave walks all heads
    if (static_cast<long>(n_slots) * runs >= 1024) {
      dim3 grid(static_cast<unsigned>((static_cast<long>(n_slots) * runs + 3) / 4));
      if (dtype == DT_BF16)
        hipLaunchKernelGGL(scores_runs_kernel<bf16_t>, grid, dim3(256), 0, st, static_cast<const bf16_t*>(v_cur),
                           static_cast<bf16_t*>(v_ref), n_slots, H, seq, dh, scores, update_ref ? 1 : 0);
      else
        hipLaunchKernelGGL(scores_runs_kernel<float>, grid, dim3(256), 0, st, static_cast<const float*>(v_cur),
                           static_cast<float*>(v_ref), n_slots, H, seq, dh, scores, update_ref ? 1 : 0);
      return hipGetLastError();
    }
  }
  const Divisor dv = make_divisor(static_cast<uint32_t>(dh));
  dim3 grid(static_cast<unsigned>((tokens + 3) / 4));
  if (dtype == DT_BF16) {
    hipLaunchKernelGGL(scores_kernel<bf16_t>, grid, dim3(256), 0, st,
                       static_cast<const bf16_t*>(v_cur), static_cast<bf16_t*>(v_ref), n_slots,
                       H, seq, dh, dv.magic, dv.shift, scores, update_ref ? 1 : 0);
  } else {
    hipLaunchKernelGGL(scores_kernel<float>, grid, dim3(256), 0, st,
                       static_cast<const float*>(v_cur), static_cast<float*>(v_ref), n_slots, H,
                       seq, dh, dv.magic, dv.shift, scores, update_ref ? 1 : 0);
  }
  return hipGetLastError();
}

hipError_t launch_select(const double* scores, int n_slots, int seq, int n, bool largest, int32_t* idx,
                         hipStream_t st) {
  if (n_slots == 0 || n == 0) return hipSuccess;
  auto kern = seq <= 64     ? select_kernel<64, 1>
              : seq <= 128  ? select_kernel<128, 1>
              : seq <= 256  ? select_kernel<256, 1>
              : seq <= 512  ? select_kernel<512, 1>
              : seq <= 1024 ? select_kernel<512, 2>
              : seq <= 2048 ? select_kernel<512, 4>
                            : select_kernel<512, 8>;
  const int threads = seq <= 64 ? 64 : seq <= 128 ? 128 : seq <= 256 ? 256 : 512;
  if (seq > 4096) return hipErrorInvalidValue;
  for (long b = 0; b < n_slots; b += kMaxGrid) {
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(std::min(kMaxGrid, n_slots - b))), dim3(threads), 0, st,
                       scores + b * seq, seq, n, largest ? 1 : 0, idx + b * n);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace marcache
