// Calibration-side kernels: min/max activation steps per K-segment (Sec. 4.3.2: s_- = |min x| / q, s_+ = max x / q;
// App. B sensitivity study: the strict min/max rule) with running maxima over calibration batches.  One pass over
// the activations, HBM-bandwidth-bound.
#include "sq_kernels.hpp"

#include <cmath>
#include <mutex>

namespace sq {

constexpr int kCalibRows = 8;   // token rows per workgroup of the unaligned form

__global__ void calib_init_kernel(float* __restrict__ amax, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) amax[i] = 0.0f;
}

// ---- the aligned pass over a batch --------------------------------------------------------------------------------------
// One workgroup of 1024 threads per compute unit, dealt to the K-segments in proportion to their width; a workgroup walks
// the 8-element chunks of its segment with a constant stride, kPassUnroll chunks per thread in flight (64 KB of bf16 per
// compute unit).  The pass is a read of X and nothing else, so what counts is bytes in flight; few, long-lived workgroups
// also keep the combining step (one atomic per workgroup and polarity on one address, ~20 ns each) off the critical path.
// 4608 x 15360 bf16 (142 MB): the maximum pass 53 -> 25 us (5.7 TB/s) and a histogram pass 78 -> 23 / 30 us against a
// thousand 256-thread workgroups of eight rows each, which exposed a memory latency per column step.
constexpr int kPassThreads = 1024;
constexpr int kPassUnroll = 4;
struct PassPlan {
  int first[SQ_MAX_SEGMENTS + 1];           // workgroups first[s] .. first[s+1] - 1 walk K-segment s
};

static PassPlan pass_plan(int M, const ActTable& tb, int K, int cus) {
  PassPlan p;
  p.first[0] = 0;
  for (int s = 0; s < tb.S; ++s) {
    const long long L = tb.kseg_off[s + 1] - tb.kseg_off[s];
    const long long chunks = (long long)M * (L / 8);
    long long n = (L * cus + K / 2) / K;                               // share of the compute units
    const long long most = (chunks + kPassThreads - 1) / kPassThreads;  // at least a chunk per thread
    n = n > most ? most : n;
    p.first[s + 1] = p.first[s] + (int)(n < 1 ? 1 : n);
  }
  return p;
}

// 8 consecutive elements as loaded
template <bool BF16> struct Chunk { v4i raw[BF16 ? 1 : 2]; };
template <bool BF16> __device__ __forceinline__ Chunk<BF16> load_chunk(const void* x, size_t e) {
  Chunk<BF16> c;
  if (BF16) {
    c.raw[0] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(x) + e));
  } else {
    c.raw[0] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const float*>(x) + e));
    c.raw[BF16 ? 0 : 1] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const float*>(x) + e + 4));
  }
  return c;
}
template <bool BF16, class F> __device__ __forceinline__ void for_each_value(const Chunk<BF16>& c, F&& take) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (BF16) {
      const uint32_t u = (uint32_t)c.raw[0][i];
      take(__uint_as_float(u << 16));
      take(__uint_as_float(u & 0xFFFF0000u));
    } else {
      take(__int_as_float(c.raw[0][i]));
      take(__int_as_float(c.raw[BF16 ? 0 : 1][i]));
    }
  }
}
// visit(chunk) for every chunk of the workgroup's share of K-segment ks
template <bool BF16, class F>
__device__ __forceinline__ void walk_segment(const void* x, int M, int K, int k0, int L, int me, int nwg, F&& visit) {
  const unsigned cpr = (unsigned)L >> 3, total = (unsigned)M * cpr, stride = (unsigned)nwg * kPassThreads;   // M K < 2^31
  const unsigned dr = stride / cpr, dc = stride - dr * cpr;
  unsigned item = (unsigned)me * kPassThreads + threadIdx.x;
  unsigned r = item / cpr, c = item - r * cpr;
  while (item < total) {
    Chunk<BF16> buf[kPassUnroll];
    bool have[kPassUnroll];
#pragma unroll
    for (int u = 0; u < kPassUnroll; ++u) {
      have[u] = item < total;
      const size_t e = have[u] ? (size_t)r * K + k0 + c * 8 : (size_t)k0;
      buf[u] = load_chunk<BF16>(x, e);
      item += stride;
      r += dr;
      c += dc;
      if (c >= cpr) { c -= cpr; ++r; }
    }
#pragma unroll
    for (int u = 0; u < kPassUnroll; ++u)
      if (have[u]) visit(buf[u]);
  }
}

// Workgroup maxima into the running ones.  Maxima are >= 0, so their fp32 bit patterns order like unsigned integers and the
// combine is an integer atomic max.  Look before combining (an uncached read): the running maximum only grows, so a value
// that already is at least this workgroup's makes the atomic unnecessary; same-address atomics serialize at ~20 ns each.
template <int WAVES>
__device__ __forceinline__ void combine_maxima(float mp, float mn, float* amax, int ks, int S) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    mp = __builtin_fmaxf(mp, __shfl_xor(mp, off, 64));
    mn = __builtin_fmaxf(mn, __shfl_xor(mn, off, 64));
  }
  __shared__ float red[2][WAVES];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[0][wave] = mp; red[1][wave] = mn; }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 1; i < WAVES; ++i) {
      mp = __builtin_fmaxf(mp, red[0][i]);
      mn = __builtin_fmaxf(mn, red[1][i]);
    }
    unsigned int* gp = reinterpret_cast<unsigned int*>(amax) + ks;
    unsigned int* gn = reinterpret_cast<unsigned int*>(amax) + S + ks;
    if (__float_as_uint(mp) > *reinterpret_cast<volatile unsigned int*>(gp)) atomicMax(gp, __float_as_uint(mp));
    if (__float_as_uint(mn) > *reinterpret_cast<volatile unsigned int*>(gn)) atomicMax(gn, __float_as_uint(mn));
  }
}

template <bool BF16>
__global__ __launch_bounds__(kPassThreads) void calib_amax_stream_kernel(const void* __restrict__ x, int M, int K, const ActTable tb,
                                                                         const PassPlan plan, float* __restrict__ amax) {
  const int b = blockIdx.x;
  int ks = 0;
  for (int s = 1; s < tb.S; ++s)
    if (b >= plan.first[s]) ks = s;
  const int k0 = tb.kseg_off[ks], L = tb.kseg_off[ks + 1] - k0;
  const bool dual = tb.dual[ks] != 0;
  float mp = 0.0f, mn = 0.0f;
  walk_segment<BF16>(x, M, K, k0, L, b - plan.first[ks], plan.first[ks + 1] - plan.first[ks], [&](const Chunk<BF16>& c) {
    for_each_value<BF16>(c, [&](float v) {
      mp = __builtin_fmaxf(mp, dual ? v : __builtin_fabsf(v));
      mn = __builtin_fmaxf(mn, dual ? -v : 0.0f);
    });
  });
  combine_maxima<kPassThreads / 64>(mp, mn, amax, ks, tb.S);
}

// Unaligned rows or segments.  grid: (row blocks, K-segments).
template <bool BF16>
__global__ __launch_bounds__(256) void calib_amax_kernel(const void* __restrict__ x, int M, int K, const ActTable tb,
                                                         float* __restrict__ amax) {
  const int ks = blockIdx.y;
  const int k0 = tb.kseg_off[ks], L = tb.kseg_off[ks + 1] - k0;
  const bool dual = tb.dual[ks] != 0;
  const int r0 = blockIdx.x * kCalibRows;
  const int nrows = (M - r0) < kCalibRows ? (M - r0) : kCalibRows;
  float mp = 0.0f, mn = 0.0f;
  for (int c = threadIdx.x; c < nrows * L; c += 256) {
    const int r = c / L, cc = c - r * L;
    const size_t e = (size_t)(r0 + r) * K + k0 + cc;
    const float v = BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(x)[e]) : reinterpret_cast<const float*>(x)[e];
    mp = __builtin_fmaxf(mp, dual ? v : __builtin_fabsf(v));
    mn = __builtin_fmaxf(mn, dual ? -v : 0.0f);
  }
  combine_maxima<4>(mp, mn, amax, ks, tb.S);
}

// steps[ks] = s_+ , steps[S + ks] = s_- : amax / 127, the neutral step 1.0 where the maximum is 0
__global__ void calib_steps_kernel(const float* __restrict__ amax, float* __restrict__ steps, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    const float a = amax[i];
    steps[i] = (a == 0.0f) ? 1.0f : a / kQmax;
  }
}

static bool pass_aligned(const void* x, int K, const ActTable& tb) {
  bool ok = (K % 8 == 0) && (reinterpret_cast<uintptr_t>(x) % 16 == 0);
  for (int s = 0; s <= tb.S; ++s) ok = ok && (tb.kseg_off[s] % 8 == 0);
  return ok;
}

hipError_t launch_calibrate_act(const void* x, bool x_is_bf16, int M, int K, const ActTable& tb, float* amax, float* steps,
                                bool accumulate, hipStream_t st) {
  const int n = 2 * tb.S;
  if (!accumulate) hipLaunchKernelGGL(calib_init_kernel, dim3(1), dim3(128), 0, st, amax, n);
  if (pass_aligned(x, K, tb)) {
    const PassPlan plan = pass_plan(M, tb, K, device_cus());
    const dim3 grid(plan.first[tb.S]);
    if (x_is_bf16) hipLaunchKernelGGL((calib_amax_stream_kernel<true>), grid, dim3(kPassThreads), 0, st, x, M, K, tb, plan, amax);
    else           hipLaunchKernelGGL((calib_amax_stream_kernel<false>), grid, dim3(kPassThreads), 0, st, x, M, K, tb, plan, amax);
  } else {
    const dim3 grid((M + kCalibRows - 1) / kCalibRows, tb.S);
    if (x_is_bf16) hipLaunchKernelGGL((calib_amax_kernel<true>), grid, dim3(256), 0, st, x, M, K, tb, amax);
    else           hipLaunchKernelGGL((calib_amax_kernel<false>), grid, dim3(256), 0, st, x, M, K, tb, amax);
  }
  hipLaunchKernelGGL(calib_steps_kernel, dim3(1), dim3(128), 0, st, amax, steps, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// Percentile clipping (App. B, dual-scale sensitivity study: p <= 0.9999 against the min/max rule).  Per K-segment
// and polarity the threshold is the nearest-rank quantile of max(x,0), max(-x,0) or |x| over the batch, zeros
// included.  The values are >= 0, so their fp32 bit patterns order like unsigned integers and the exact order
// statistic comes from a radix select on those bits, most significant digit first: a histogram pass over the
// activations per digit (one pass per 8 bits: two for bf16 inputs, four for fp32), each followed by a tiny kernel
// that walks the 256 bins from the top, picks the bin holding the wanted rank and narrows the search to it.
// Digit 0 is never counted (it would make the zeros of the other polarity one hot bin): its count is the rest of
// the bucket.
// ------------------------------------------------------------------------------------------------------------
struct PctState {                                 // the caller's workspace
  unsigned int hist[SQ_MAX_SEGMENTS][2][256];     // [ks][polarity][digit], zero between passes
  unsigned int rank[SQ_MAX_SEGMENTS][2];          // wanted rank from the top (1 = largest) inside the bucket
  unsigned int bucket[SQ_MAX_SEGMENTS][2];        // elements that share the prefix found so far
  unsigned int prefix[SQ_MAX_SEGMENTS][2];        // magnitude bits found so far
};
struct PctRanks {                                 // per K-segment: elements of a batch, rank from the top
  unsigned int n[SQ_MAX_SEGMENTS];
  unsigned int r[SQ_MAX_SEGMENTS];
};

// copies of every histogram bin in LDS, consecutive (so in different banks), one per lane class: activations put a third of
// a wave's lanes on one exponent bin, and same-address LDS atomics serialize
constexpr int kPctCopies = 8;           // unaligned form
constexpr int kPctStreamCopies = 32;    // 64 KB: one workgroup per compute unit

size_t calibrate_workspace_bytes() { return sizeof(PctState); }

__global__ void pct_init_kernel(PctState* __restrict__ st, const PctRanks rk, int S) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < S * 2 * 256) (&st->hist[0][0][0])[i] = 0u;
  if (i < S * 2) {
    const int ks = i >> 1, pol = i & 1;
    st->rank[ks][pol] = rk.r[ks];
    st->bucket[ks][pol] = rk.n[ks];
    st->prefix[ks][pol] = 0u;
  }
}

// Counts digit (bits >> shift) & dmask of every value whose bits above the digit (himask) equal the prefix found so far.
template <int COPIES>
struct DigitCounter {
  unsigned int (*h)[256][COPIES];           // LDS [2][256][COPIES]
  unsigned int pre_p, pre_n, dmask, himask;
  int shift, copy;
  bool dual;
  __device__ __forceinline__ void count(int pol, unsigned int bits, unsigned int pre) const {
    if ((bits & himask) == pre) {
      const unsigned int d = (bits >> shift) & dmask;
      if (d != 0u) atomicAdd(&h[pol][d][copy], 1u);
    }
  }
  __device__ __forceinline__ void take(float v) const {
    const unsigned int bits = __float_as_uint(v), mag = bits & 0x7FFFFFFFu;
    if (dual) {                             // a value counts on the side of its sign only: digit 0 is never counted, and the
      const bool ng = v < 0.0f;             // other side's zero has no other digit to match with
      if (ng || v > 0.0f) count(ng ? 1 : 0, mag, ng ? pre_n : pre_p);
    } else {
      count(0, mag, pre_p);
    }
  }
};

template <int COPIES, int THREADS>
__device__ __forceinline__ void flush_histogram(const unsigned int (*h)[256][COPIES], PctState* st, int ks) {
  for (int i = threadIdx.x; i < 512; i += THREADS) {
    const int pol = i >> 8, d = i & 255;
    unsigned int c = 0u;
    for (int k = 0; k < COPIES; ++k) c += h[pol][d][(k + i) % COPIES];   // neighbouring bins start on different banks
    if (c != 0u) atomicAdd(&st->hist[ks][pol][d], c);
  }
}

// The two digits of a bf16 pattern, counted on the pattern itself: sign and exponent are its top nine bits, so the first
// pass is one bit-field extract, one address and one LDS atomic per value (the general take() is 15 instructions, as much
// time as the atomics: 58 us a pass on 4608 x 15360 against 23 us for the first pass, a read at 6.1 TB/s, and 30 for the second
// this way), the second one compares them with the two prefixes and counts the mantissa.  Digit 0 is counted along (the select
// kernel does not look at it).  A chunk with a pattern above infinity (NaN: inputs must be finite) takes the general route, which
// passes it over in a polarity-split segment and counts it under its magnitude in a one-step segment.
typedef unsigned short v2us __attribute__((ext_vector_type(2)));
template <bool FIRST, bool DUAL, int COPIES>
__device__ __forceinline__ void count_bf16(const Chunk<true>& c, const DigitCounter<COPIES>& dc, unsigned int* own,
                                           const unsigned int key_p, const unsigned int key_n) {
  v2us top = (v2us)(0);
#pragma unroll
  for (int i = 0; i < 4; ++i) top = __builtin_elementwise_max(top, __builtin_bit_cast(v2us, (uint32_t)c.raw[0][i] & 0x7FFF7FFFu));
  if (top[0] > 0x7F80 || top[1] > 0x7F80) {
    for_each_value<true>(c, [&](float v) { dc.take(v); });
    return;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t u = (uint32_t)c.raw[0][i >> 1];
    const int lo = (i & 1) ? 16 : 0;
    const uint32_t key = (u >> (lo + 7)) & (DUAL ? 0x1FFu : 0xFFu);             // [sign] exponent
    if (FIRST) {
      atomicAdd(own + key * COPIES, 1u);
    } else if (key == key_p || (DUAL && key == key_n)) {
      atomicAdd(own + ((DUAL ? key & 0x100u : 0u) | ((u >> lo) & 0x7Fu)) * COPIES, 1u);
    }
  }
}

template <bool BF16>
__global__ __launch_bounds__(kPassThreads) void pct_hist_stream_kernel(const void* __restrict__ x, int M, int K, const ActTable tb,
                                                                       const PassPlan plan, PctState* __restrict__ st, int shift,
                                                                       unsigned int dmask, unsigned int himask) {
  const int b = blockIdx.x;
  int ks = 0;
  for (int s = 1; s < tb.S; ++s)
    if (b >= plan.first[s]) ks = s;
  const int k0 = tb.kseg_off[ks], L = tb.kseg_off[ks + 1] - k0;
  __shared__ unsigned int h[2][256][kPctStreamCopies];
  for (int i = threadIdx.x; i < 2 * 256 * kPctStreamCopies; i += kPassThreads) (&h[0][0][0])[i] = 0u;
  const DigitCounter<kPctStreamCopies> dc{h, st->prefix[ks][0], st->prefix[ks][1], dmask, himask, shift,
                                          (int)threadIdx.x & (kPctStreamCopies - 1), tb.dual[ks] != 0};
  __syncthreads();
  auto walk = [&](auto&& visit) { walk_segment<BF16>(x, M, K, k0, L, b - plan.first[ks], plan.first[ks + 1] - plan.first[ks], visit); };
  if constexpr (BF16) {
    unsigned int* own = &h[0][0][dc.copy];
    const unsigned int key_p = dc.pre_p >> 23, key_n = 0x100u | (dc.pre_n >> 23);
    const bool first = himask == 0u;
    if (first && dc.dual) walk([&](const Chunk<BF16>& c) { count_bf16<true, true>(c, dc, own, key_p, key_n); });
    else if (first) walk([&](const Chunk<BF16>& c) { count_bf16<true, false>(c, dc, own, key_p, key_n); });
    else if (dc.dual) walk([&](const Chunk<BF16>& c) { count_bf16<false, true>(c, dc, own, key_p, key_n); });
    else walk([&](const Chunk<BF16>& c) { count_bf16<false, false>(c, dc, own, key_p, key_n); });
  } else {
    walk([&](const Chunk<BF16>& c) { for_each_value<BF16>(c, [&](float v) { dc.take(v); }); });
  }
  __syncthreads();
  flush_histogram<kPctStreamCopies, kPassThreads>(h, st, ks);
}

// Unaligned rows or segments.  grid: (row blocks, K-segments).
template <bool BF16>
__global__ __launch_bounds__(256) void pct_hist_kernel(const void* __restrict__ x, int M, int K, const ActTable tb,
                                                       PctState* __restrict__ st, int shift, unsigned int dmask,
                                                       unsigned int himask) {
  const int ks = blockIdx.y;
  const int k0 = tb.kseg_off[ks], L = tb.kseg_off[ks + 1] - k0;
  const int r0 = blockIdx.x * kCalibRows;
  const int nrows = (M - r0) < kCalibRows ? (M - r0) : kCalibRows;
  __shared__ unsigned int h[2][256][kPctCopies];
  for (int i = threadIdx.x; i < 2 * 256 * kPctCopies; i += 256) (&h[0][0][0])[i] = 0u;
  const DigitCounter<kPctCopies> dc{h, st->prefix[ks][0], st->prefix[ks][1], dmask, himask, shift,
                                    (int)threadIdx.x & (kPctCopies - 1), tb.dual[ks] != 0};
  __syncthreads();
  for (int c = threadIdx.x; c < nrows * L; c += 256) {
    const int r = c / L, cc = c - r * L;
    const size_t e = (size_t)(r0 + r) * K + k0 + cc;
    dc.take(BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(x)[e]) : reinterpret_cast<const float*>(x)[e]);
  }
  __syncthreads();
  flush_histogram<kPctCopies, 256>(h, st, ks);
}

// One 256-thread workgroup per (K-segment, polarity): suffix sums of the 256 bins from the top (a log-step scan in
// LDS); the bin d >= 1 whose suffix sum first reaches the wanted rank holds it, else it lies in the uncounted digit 0.
// The bucket is narrowed to that bin and the histogram cleared for the next pass.  After the last digit the prefix is
// the threshold: fold it into the running maxima and write the steps (amax, steps: [2][S], as the min/max calibration).
__global__ __launch_bounds__(256) void pct_select_kernel(PctState* __restrict__ st, int S, int shift, int last, int accumulate,
                                                         float* __restrict__ amax, float* __restrict__ steps) {
  const int i = blockIdx.x;                                  // grid: 2 S
  const int pol = i / S, ks = i - pol * S;
  const int d = threadIdx.x;
  unsigned int* h = st->hist[ks][pol];
  __shared__ unsigned int suf[256];
  const unsigned int own = d >= 1 ? h[d] : 0u;               // digit 0 is not counted
  h[d] = 0u;
  suf[d] = own;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {                  // suf[d] = sum of bins d .. 255
    const unsigned int add = d + off < 256 ? suf[d + off] : 0u;
    __syncthreads();
    suf[d] += add;
    __syncthreads();
  }
  const unsigned int r = st->rank[ks][pol], bucket = st->bucket[ks][pol], pre = st->prefix[ks][pol];
  const unsigned int above = d < 255 ? suf[d + 1] : 0u;      // elements in bins above d
  const unsigned int total = suf[1];                         // all counted elements (bins 1 .. 255)
  __syncthreads();
  // exactly one thread holds the rank: bin d >= 1 with above < r <= above + own, or d == 0 when r > total
  const bool mine = d >= 1 ? (above < r && r <= above + own) : (r > total);
  if (mine) {
    const unsigned int taken = d >= 1 ? above : total;
    const unsigned int npre = pre | ((unsigned int)d << shift);
    st->rank[ks][pol] = r - taken;
    st->bucket[ks][pol] = d >= 1 ? own : bucket - total;
    st->prefix[ks][pol] = npre;
    if (last) {
      const float t = __uint_as_float(npre);
      float a = accumulate ? amax[i] : 0.0f;
      a = __builtin_fmaxf(a, t);
      amax[i] = a;
      steps[i] = (a == 0.0f) ? 1.0f : a / kQmax;
    }
  }
}

hipError_t launch_calibrate_act_percentile(const void* x, bool x_is_bf16, int M, int K, const ActTable& tb, double p,
                                           float* amax, float* steps, void* workspace, bool accumulate, hipStream_t st) {
  PctState* ws = reinterpret_cast<PctState*>(workspace);
  PctRanks rk;
  for (int s = 0; s < tb.S; ++s) {
    const long long n = (long long)M * (tb.kseg_off[s + 1] - tb.kseg_off[s]);
    long long k = (long long)std::ceil(p * (double)n);      // nearest rank, in IEEE double
    k = k < 1 ? 1 : (k > n ? n : k);
    rk.n[s] = (unsigned int)n;
    rk.r[s] = (unsigned int)(n - k + 1);                    // k-th smallest = (n - k + 1)-th largest
  }
  const int nclear = tb.S * 2 * 256;
  hipLaunchKernelGGL(pct_init_kernel, dim3((nclear + 255) / 256), dim3(256), 0, st, ws, rk, tb.S);
  const bool vec = pass_aligned(x, K, tb);
  const PassPlan plan = pass_plan(M, tb, K, device_cus());
  const dim3 grid((M + kCalibRows - 1) / kCalibRows, tb.S);
  // digits of the magnitude bits, most significant first; a bf16 value has nothing below bit 16
  static const int kShift[4] = {23, 15, 7, 0};
  static const unsigned int kMask[4] = {0xFFu, 0xFFu, 0xFFu, 0x7Fu};
  const int npass = x_is_bf16 ? 2 : 4;
  for (int ps = 0; ps < npass; ++ps) {
    int shift = kShift[ps];
    unsigned int dmask = kMask[ps];
    if (x_is_bf16 && ps == 1) { shift = 16; dmask = 0x7Fu; }
    const unsigned int himask = 0x7FFFFFFFu & ~((dmask << shift) | ((1u << shift) - 1u));
#define SQ_PCT(B) \
  if (vec) hipLaunchKernelGGL((pct_hist_stream_kernel<B>), dim3(plan.first[tb.S]), dim3(kPassThreads), 0, st, x, M, K, tb, plan, ws, shift, dmask, himask); \
  else hipLaunchKernelGGL((pct_hist_kernel<B>), grid, dim3(256), 0, st, x, M, K, tb, ws, shift, dmask, himask)
    if (x_is_bf16) { SQ_PCT(true); }
    else           { SQ_PCT(false); }
#undef SQ_PCT
    hipLaunchKernelGGL(pct_select_kernel, dim3(2 * tb.S), dim3(256), 0, st, ws, tb.S, shift,
                       ps == npass - 1 ? 1 : 0, accumulate ? 1 : 0, amax, steps);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------------------
// The same calibration for callers that cannot allocate or pass a workspace (HIP graph capture, serving loops,
// harnesses that forbid hipMalloc): the radix-select state lives in a file-scope device array.  Every device the
// library runs on holds its own copy of the array at its own address; the address is looked up once per device
// (with that device current) and used from then on — the array's name is a host-side stand-in, never a device
// address.  All calls on one device share the array: calls that overlap on a device race.  Nothing has to be zero
// on entry: pct_init_kernel clears the histograms and sets ranks, buckets and prefixes at the start of every call.
// ------------------------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[sizeof(PctState)];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_lock;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

size_t calibrate_static_scratch_bytes() { return sizeof(PctState); }

hipError_t launch_calibrate_act_percentile_static(const void* x, bool x_is_bf16, int M, int K, const ActTable& tb, double p,
                                                  float* amax, float* steps, bool accumulate, hipStream_t st) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void* ptr = nullptr;
  {
    std::lock_guard<std::mutex> guard(g_scratch_lock);
    if (g_scratch_ptr[dev] == nullptr) {
      void* found = nullptr;
      e = hipGetSymbolAddress(&found, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      if (found == nullptr) return hipErrorInvalidSymbol;
      g_scratch_ptr[dev] = found;
    }
    ptr = g_scratch_ptr[dev];
  }
  return launch_calibrate_act_percentile(x, x_is_bf16, M, K, tb, p, amax, steps, ptr, accumulate, st);
}

}  // namespace sq
