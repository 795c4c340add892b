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

__device__ __forceinline__ float step_of(float a) { return (a == 0.0f) ? 1.0f : a / kQmax; }   // the neutral step where the maximum is 0

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

// steps[ks] = s_+ , steps[S + ks] = s_-
__global__ void calib_steps_kernel(const float* __restrict__ amax, float* __restrict__ steps, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) steps[i] = step_of(amax[i]);
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
// activations per digit (one pass per 8 bits: two for bf16 inputs, four for fp32), after which the bin of the 256 that
// holds the wanted rank is searched from the top and the search narrowed to it.  Digit 0 is never counted (it would make
// the zeros of the other polarity one hot bin): its count is the rest of the bucket.
// Aligned bf16 batches need one pass as a rule: a sample of the segment says about where the order statistic lies, and a
// pass counts the 254 bit patterns around that place (a factor of two to either side) one by one, with everything above in one
// more bin.  Where the rank falls outside, the two digit passes follow; else they return at once.  4608 x 15360 (142 MB),
// p = 0.9999, kernels: 5.4 us sample, 26.6 window pass, 4.8 search, 2 x 4.8 passes with nothing to do, against 4.8 clearing,
// 23 + 30 digit passes, 2 x 4.8 searches; with both weight formats and the min/max calibration 183.2 -> 163.2 us.
// The call alone, digit passes only / window / window missed: 4608 x 15360 61 / 37 / 90 - 95 us, 1024 x 4608 20 - 24 / 19 / 35 - 43,
// 256 x 1152 15.5 / 14.7 / 20 - 26.  Normal values, GELU outputs and a channel in a hundred ten times as strong are found for p from
// 0.9 to 0.9999, the first two also beyond.  Missed are: NaN in a polarity-split segment; tails without a scale from p = 0.9999 on
// (Cauchy, lognormal of sigma 2, a channel in a thousand a hundred times as strong), p = 1 of strong channels and of Student's t with
// three degrees; in a polarity-split segment a p that is the share of the other sign's values, at which the quantile is next to the
// zeros (p = 0.5 of symmetric values).  A test of the sample's spread that sends such segments on the digit passes at once took 76 -
// 81 us and 31 - 36 there, as the searches behind passes with work cost more, and sent Cauchy at p = 0.999 there too (37 / 19 now).
// ------------------------------------------------------------------------------------------------------------
struct PctState {                                 // the caller's workspace
  unsigned int hist[SQ_MAX_SEGMENTS][2][256];     // [ks][polarity][digit], zero between passes; digit 0 is no count: [ks][0][0]
                                                  // counts the workgroups that have finished the segment's pass, [ks][1][0]
                                                  // is set where the window pass has met NaN
  unsigned int rank[SQ_MAX_SEGMENTS][2];          // wanted rank from the top (1 = largest) inside the bucket
  unsigned int open[SQ_MAX_SEGMENTS][2];          // 0: the threshold is found
  unsigned int prefix[SQ_MAX_SEGMENTS][2];        // magnitude bits found so far; window pass: bf16 pattern of its bin 0
};
struct PctRanks {                                 // per K-segment: rank from the top in the batch
  unsigned int r[SQ_MAX_SEGMENTS];
};

// copies of every histogram bin in LDS, consecutive (so in different banks), one per lane class: activations put a third of
// a wave's lanes on one exponent bin, and same-address LDS atomics serialize
constexpr int kPctCopies = 8;           // unaligned form
constexpr int kPctStreamCopies = 32;    // 64 KB: one workgroup per compute unit

size_t calibrate_workspace_bytes() { return sizeof(PctState); }

// True in the workgroup that is the last of n to arrive at a counter that was 0 before the launch.  Called by one thread after the
// workgroup's atomics have completed (each wave waits for its own, then the workgroup's barrier); what other workgroups
// added by agent-scope atomics before they arrived can then be read with agent-scope loads.
__device__ __forceinline__ bool arrive_last(unsigned int* counter, unsigned int n) {
  return __hip_atomic_fetch_add(counter, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u == n;
}
// One workgroup of 1024 threads per K-segment clears its state.  SAMPLE (aligned bf16): it also reads up to kPctSample chunks,
// spread evenly over the segment with a jitter inside each share (a plain stride could walk one column of every row), and
// centres the window on the sample's order statistic, found to half a binade.  1024 chunks = 8192 values: more of them cost
// more (a compute unit's histogram atomics) than the place gains by.
constexpr unsigned kPctSample = 1024;
constexpr unsigned kPctWindowHalf = 127, kPctBaseMax = 0x7F00;
template <bool SAMPLE>
__global__ __launch_bounds__(kPassThreads) void pct_init_kernel(const void* __restrict__ x, int M, int K, const ActTable tb,
                                                                PctState* __restrict__ st, const PctRanks rk) {
  const int ks = blockIdx.x, t = threadIdx.x;
  if (t < 512) (&st->hist[ks][0][0])[t] = 0u;
  if (t < 2) {
    st->rank[ks][t] = rk.r[ks];
    st->open[ks][t] = 1u;
    st->prefix[ks][t] = 0u;
  }
  if constexpr (SAMPLE) {
    constexpr int COPIES = 4;
    __shared__ unsigned int h[2][512][COPIES];                // bins of half a binade: pattern >> 6
    __shared__ unsigned int wave_sum[16];
    for (int i = t; i < 2 * 512 * COPIES; i += kPassThreads) (&h[0][0][0])[i] = 0u;
    __syncthreads();
    const bool dual = tb.dual[ks] != 0;
    const int k0 = tb.kseg_off[ks];
    const unsigned cpr = (unsigned)(tb.kseg_off[ks + 1] - k0) >> 3, total = (unsigned)M * cpr;
    const unsigned ns = total < kPctSample ? total : kPctSample;
    const unsigned share = total / ns;
    for (unsigned j = t; j < ns; j += kPassThreads) {
      const unsigned first = (unsigned)((unsigned long long)j * total / ns);
      const unsigned item = first + ((j * 2654435761u) >> 8) % share;
      const unsigned r = item / cpr, c = item - r * cpr;
      const v4i raw = *reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(x) + (size_t)r * K + k0 + c * 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const unsigned u = ((unsigned)raw[i >> 1] >> (i & 1 ? 16 : 0)) & 0xFFFFu;
        atomicAdd(&h[dual ? u >> 15 : 0][(u & 0x7FFFu) >> 6][t & (COPIES - 1)], 1u);
      }
    }
    __syncthreads();
    // thread (polarity, d): elements of the bins d .. 511, by a scan from the top inside each wave and over the eight waves
    const int pol = t >> 9, d = 511 - (t & 511), lane = t & 63, wave = t >> 6;
    unsigned own = 0u;
    for (int k = 0; k < COPIES; ++k) own += h[pol][d][k];
    own = d != 0 ? own : 0u;
    unsigned suf = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned up = (unsigned)__shfl_up((int)suf, off, 64);
      suf += lane >= off ? up : 0u;
    }
    if (lane == 63) wave_sum[wave] = suf;
    __syncthreads();
    for (int w = pol * 8; w < wave; ++w) suf += wave_sum[w];
    const unsigned want = (unsigned)((unsigned long long)rk.r[ks] * ns / total), rs = want < 1u ? 1u : want;
    if (d != 0 && suf - own < rs && rs <= suf) {              // no thread: the rank is among the smallest, the window starts at 0
      const int base = (d << 6) + 32 - (int)kPctWindowHalf;
      st->prefix[ks][pol] = base < 0 ? 0u : base > (int)kPctBaseMax ? kPctBaseMax : (unsigned)base;
    }
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
    if (d != 0 && c != 0u) atomicAdd(&st->hist[ks][pol][d], c);
  }
}

// The search after a pass, by one workgroup of at least 512 threads: thread (polarity, d) holds bin d; suffix sums of the 256 bins
// from the top (a log-step scan in LDS); the bin d >= 1 whose suffix sum first reaches the wanted rank holds it, else it lies in
// the uncounted digit 0.  The bucket is narrowed to that bin and the histogram cleared for the next pass.  When the
// threshold is found (the prefix after the last digit, or the pattern base + d of a window; its bins 0 and 255 are open ends,
// except that below base 0 there are only zeros) it is folded into the running maxima and the steps are written (amax,
// steps: [2][S], as the min/max calibration).
enum PctPass { PCT_DIGIT, PCT_LAST_DIGIT, PCT_WINDOW };
__device__ __forceinline__ void pct_select(PctState* st, int ks, int S, int shift, PctPass pass, int accumulate, float* amax, float* steps,
                                           unsigned int (*suf)[256]) {
  const int pol = (threadIdx.x >> 8) & 1, d = threadIdx.x & 255;
  const bool in = threadIdx.x < 512;
  unsigned int own = 0u;
  bool nan = false;
  if (in) {
    if (d != 0) own = __hip_atomic_load(&st->hist[ks][pol][d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    nan = __hip_atomic_load(&st->hist[ks][1][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
  }
  __syncthreads();
  if (in) {
    st->hist[ks][pol][d] = 0u;                               // digit 0: the counter of finished workgroups
    suf[pol][d] = own;
  }
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {                  // suf[d] = sum of bins d .. 255
    const unsigned int add = in && d + off < 256 ? suf[pol][d + off] : 0u;
    __syncthreads();
    if (in) suf[pol][d] += add;
    __syncthreads();
  }
  const bool open = in && st->open[ks][pol] != 0u;
  const unsigned int r = st->rank[ks][pol], pre = st->prefix[ks][pol];
  const unsigned int above = d < 255 ? suf[pol][d + 1] : 0u; // elements in bins above d
  const unsigned int total = suf[pol][1];                    // all counted elements (bins 1 .. 255)
  // exactly one thread holds the rank: bin d >= 1 with above < r <= above + own, or d == 0 when r > total
  const bool mine = d >= 1 ? (above < r && r <= above + own) : (r > total);
  __syncthreads();                                           // every thread has read the state before it changes
  if (open && mine) {
    bool found = pass == PCT_LAST_DIGIT;
    unsigned int bits = pre | ((unsigned int)d << shift);
    if (pass == PCT_WINDOW) {
      found = !nan && (d == 0 ? pre == 0u : d < 255);
      bits = found ? (pre + (unsigned int)d) << 16 : 0u;
    } else {
      st->rank[ks][pol] = r - (d >= 1 ? above : total);
    }
    st->prefix[ks][pol] = bits;
    if (found) {
      const int i = pol * S + ks;
      const float a = __builtin_fmaxf(accumulate ? amax[i] : 0.0f, __uint_as_float(bits));
      st->open[ks][pol] = 0u;
      amax[i] = a;
      steps[i] = step_of(a);
    }
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

// The window pass: bf16 patterns base .. base + 255 one bin each, in packed 16-bit arithmetic (two values per instruction).  With
// two polarities a pattern's distance above its own base (saturated: 0 below it) is 0 on the side of the other sign, whose
// patterns lie below sign bit + base once the sign bit is where the side's own patterns have it; the difference of the two,
// clamped to -255 .. 255, names the bin.  Bin 0 is counted along (in its own bank per lane class, which is cheaper than a
// branch).  top collects the largest magnitude pattern for the test for NaN behind the pass.
template <bool DUAL, int COPIES>
__device__ __forceinline__ void count_window(const Chunk<true>& c, char* lds, const v2us at, const v2us base_p, const v2us base_n, v2us& top) {
  typedef short v2s __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t u = (uint32_t)c.raw[0][i];
    const v2us mag = __builtin_bit_cast(v2us, u & 0x7FFF7FFFu);
    v2s d;
    if (DUAL) {
      top = __builtin_elementwise_max(top, mag);
      d = __builtin_bit_cast(v2s, __builtin_elementwise_sub_sat(__builtin_bit_cast(v2us, u ^ 0x80008000u), base_p) -
                                      __builtin_elementwise_sub_sat(__builtin_bit_cast(v2us, u), base_n));
      d = __builtin_elementwise_max(d, (v2s)(short)-255);
    } else {
      d = __builtin_bit_cast(v2s, __builtin_elementwise_sub_sat(mag, base_p));
    }
    d = __builtin_elementwise_min(d, (v2s)(short)255);
    const uint32_t to = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2us, d) * (unsigned short)(COPIES * 4) + at);   // byte offsets
    atomicAdd(reinterpret_cast<unsigned int*>(lds + (to & 0xFFFFu)), 1u);
    atomicAdd(reinterpret_cast<unsigned int*>(lds + (to >> 16)), 1u);
  }
}

// One pass over the batch.  WINDOW: the pass around the sampled place.  The search behind a pass is a kernel of its own (4.8 us in a
// trace, about half of it in a stream of launches) except behind the digit passes of bf16 batches, which as a rule have
// nothing to do: there the last workgroup of a K-segment searches, so that they are two launches that return at once and not four.
// Where the pass runs that costs more (the arrivals' fences and the search: 8 us behind the window pass).
template <bool BF16, bool WINDOW>
__global__ __launch_bounds__(kPassThreads) void pct_hist_stream_kernel(const void* __restrict__ x, int M, int K, const ActTable tb,
                                                                       const PassPlan plan, PctState* __restrict__ st, int shift,
                                                                       unsigned int dmask, unsigned int himask, PctPass pass,
                                                                       int accumulate, float* __restrict__ amax, float* __restrict__ steps) {
  const int b = blockIdx.x;
  int ks = 0;
  for (int s = 1; s < tb.S; ++s)
    if (b >= plan.first[s]) ks = s;
  if ((st->open[ks][0] | st->open[ks][1]) == 0u) return;     // written by an earlier launch, the same for all of the segment
  const int k0 = tb.kseg_off[ks], L = tb.kseg_off[ks + 1] - k0;
  const unsigned nwg = (unsigned)(plan.first[ks + 1] - plan.first[ks]);
  const bool dual = tb.dual[ks] != 0;
  __shared__ unsigned int h[2][256][kPctStreamCopies];
  __shared__ unsigned int suf[2][256];
  __shared__ bool last;
  for (int i = threadIdx.x; i < 2 * 256 * kPctStreamCopies; i += kPassThreads) (&h[0][0][0])[i] = 0u;
  __syncthreads();
  auto walk = [&](auto&& visit) { walk_segment<BF16>(x, M, K, k0, L, b - plan.first[ks], (int)nwg, visit); };
  unsigned int* own = &h[0][0][threadIdx.x & (kPctStreamCopies - 1)];
  if constexpr (WINDOW) {
    static_assert(sizeof(h) <= 65536, "16-bit byte offsets");
    char* lds = reinterpret_cast<char*>(&h[0][0][0]);
    const v2us at = (v2us)(unsigned short)((255 * kPctStreamCopies + ((int)threadIdx.x & (kPctStreamCopies - 1))) * 4);
    const v2us bp = (v2us)(unsigned short)((dual ? 0x8000u : 0u) + st->prefix[ks][0]), bn = (v2us)(unsigned short)(0x8000u + st->prefix[ks][1]);
    v2us top = (v2us)(0);
    if (dual) walk([&](const Chunk<true>& c) { count_window<true, kPctStreamCopies>(c, lds, at, bp, bn, top); });
    else walk([&](const Chunk<true>& c) { count_window<false, kPctStreamCopies>(c, lds, at, bp, bn, top); });
    // NaN counts in neither polarity: the digit passes sort it out, for which this pass must not find the rank
    if (top[0] > 0x7F80 || top[1] > 0x7F80) atomicOr(&st->hist[ks][1][0], 1u);
    __syncthreads();
    if (threadIdx.x < 512) {
      const int pol = threadIdx.x >> 8, d = threadIdx.x & 255, bin = 255 + (pol ? -d : d);
      unsigned int n = 0u;
      for (int k = 0; k < kPctStreamCopies; ++k) n += (&h[0][0][0])[bin * kPctStreamCopies + ((k + bin) & (kPctStreamCopies - 1))];
      if (d != 0 && n != 0u) atomicAdd(&st->hist[ks][pol][d], n);
    }
  } else {
    const DigitCounter<kPctStreamCopies> dc{h, st->prefix[ks][0], st->prefix[ks][1], dmask, himask, shift,
                                            (int)threadIdx.x & (kPctStreamCopies - 1), dual};
    if constexpr (BF16) {
      const unsigned int key_p = dc.pre_p >> 23, key_n = 0x100u | (dc.pre_n >> 23);
      const bool first = himask == 0u;
      if (first && dual) walk([&](const Chunk<BF16>& c) { count_bf16<true, true>(c, dc, own, key_p, key_n); });
      else if (first) walk([&](const Chunk<BF16>& c) { count_bf16<true, false>(c, dc, own, key_p, key_n); });
      else if (dual) walk([&](const Chunk<BF16>& c) { count_bf16<false, true>(c, dc, own, key_p, key_n); });
      else walk([&](const Chunk<BF16>& c) { count_bf16<false, false>(c, dc, own, key_p, key_n); });
    } else {
      walk([&](const Chunk<BF16>& c) { for_each_value<BF16>(c, [&](float v) { dc.take(v); }); });
    }
    __syncthreads();
    flush_histogram<kPctStreamCopies, kPassThreads>(h, st, ks);
  }
  if (WINDOW || !BF16) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this wave's counts are in
  __syncthreads();
  if (threadIdx.x == 0) last = arrive_last(&st->hist[ks][0][0], nwg);
  __syncthreads();
  if (last) pct_select(st, ks, tb.S, shift, pass, accumulate, amax, steps, suf);
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

__global__ __launch_bounds__(512) void pct_select_kernel(PctState* __restrict__ st, int S, int shift, PctPass pass, int accumulate,
                                                         float* __restrict__ amax, float* __restrict__ steps) {
  __shared__ unsigned int suf[2][256];
  pct_select(st, blockIdx.x, S, shift, pass, accumulate, amax, steps, suf);
}

hipError_t launch_calibrate_act_percentile(const void* x, bool x_is_bf16, int M, int K, const ActTable& tb, double p,
                                           float* amax, float* steps, void* workspace, bool accumulate, hipStream_t st) {
  PctState* ws = reinterpret_cast<PctState*>(workspace);
  PctRanks rk;
  for (int s = 0; s < tb.S; ++s) {
    const long long n = (long long)M * (tb.kseg_off[s + 1] - tb.kseg_off[s]);
    long long k = (long long)std::ceil(p * (double)n);      // nearest rank, in IEEE double
    k = k < 1 ? 1 : (k > n ? n : k);
    rk.r[s] = (unsigned int)(n - k + 1);                    // k-th smallest = (n - k + 1)-th largest
  }
  const bool vec = pass_aligned(x, K, tb);
  const PassPlan plan = pass_plan(M, tb, K, device_cus());
  const dim3 grid((M + kCalibRows - 1) / kCalibRows, tb.S);
  const int acc = accumulate ? 1 : 0;
  if (vec && x_is_bf16) {
    hipLaunchKernelGGL((pct_init_kernel<true>), dim3(tb.S), dim3(kPassThreads), 0, st, x, M, K, tb, ws, rk);
    hipLaunchKernelGGL((pct_hist_stream_kernel<true, true>), dim3(plan.first[tb.S]), dim3(kPassThreads), 0, st, x, M, K, tb, plan, ws,
                       0, 0u, 0u, PCT_WINDOW, acc, amax, steps);
    hipLaunchKernelGGL(pct_select_kernel, dim3(tb.S), dim3(512), 0, st, ws, tb.S, 0, PCT_WINDOW, acc, amax, steps);
  } else {
    hipLaunchKernelGGL((pct_init_kernel<false>), dim3(tb.S), dim3(kPassThreads), 0, st, x, M, K, tb, ws, rk);
  }
  // digits of the magnitude bits, most significant first; a bf16 value has nothing below bit 16
  static const int kShift[4] = {23, 15, 7, 0};
  static const unsigned int kMask[4] = {0xFFu, 0xFFu, 0xFFu, 0x7Fu};
  const int npass = x_is_bf16 ? 2 : 4;
  for (int ps = 0; ps < npass; ++ps) {
    int shift = kShift[ps];
    unsigned int dmask = kMask[ps];
    if (x_is_bf16 && ps == 1) { shift = 16; dmask = 0x7Fu; }
    const unsigned int himask = 0x7FFFFFFFu & ~((dmask << shift) | ((1u << shift) - 1u));
    const PctPass pass = ps == npass - 1 ? PCT_LAST_DIGIT : PCT_DIGIT;
#define SQ_PCT(B) \
  if (vec) \
    hipLaunchKernelGGL((pct_hist_stream_kernel<B, false>), dim3(plan.first[tb.S]), dim3(kPassThreads), 0, st, x, M, K, tb, plan, ws, shift, \
                       dmask, himask, pass, acc, amax, steps); \
  else \
    hipLaunchKernelGGL((pct_hist_kernel<B>), grid, dim3(256), 0, st, x, M, K, tb, ws, shift, dmask, himask)
    if (x_is_bf16) { SQ_PCT(true); }
    else           { SQ_PCT(false); }
#undef SQ_PCT
    if (!vec || !x_is_bf16) hipLaunchKernelGGL(pct_select_kernel, dim3(tb.S), dim3(512), 0, st, ws, tb.S, shift, pass, acc, amax, steps);
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
