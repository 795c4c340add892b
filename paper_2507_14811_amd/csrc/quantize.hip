// Quant(.) kernels: the fused polarity-split / DualScale activation quantizer (Sec. 4.3.2) and the
// per-segment symmetric weight quantizer (Sec. 3 quantizer applied per segment, Sec. 4.2.2).
// Both are single-pass, HBM-bandwidth-bound streams.
#include "sq_kernels.hpp"

#include <cmath>

namespace sq {

// ------------------------------------------------------------------------------------------------
// Activation quantize.  Output: one int8 code per element, X^ = X^_+ + X^_- ("polarity-merged"): in a
// DualScale K-segment the element went through the s_+ branch of Q_dual when x >= 0 (code >= 0) and
// through the s_- branch when x < 0 (code <= 0), so X^_+ = max(X^, 0) and X^_- = min(X^, 0) are recovered
// exactly from the sign; in a single-scale segment the code is the symmetric one.
//
// Fast path: K and every K-segment boundary are multiples of 16, so a thread owns 16 consecutive elements
// of one row and one segment: 32 B (bf16) or 64 B (fp32) in, 16 B out, one chunk per thread (kActUnroll).
// ------------------------------------------------------------------------------------------------
constexpr int kActUnroll = 1;     // measured on the headline layer: 37.4 us with 1, 39.6 with 2, 44 with 4, 52.6 with 8 chunks per thread
constexpr int kActChunk = 16;

__device__ __forceinline__ uint32_t pack4(int c0, int c1, int c2, int c3) {
  return (uint32_t)(c0 & 0xFF) | ((uint32_t)(c1 & 0xFF) << 8) | ((uint32_t)(c2 & 0xFF) << 16) | ((uint32_t)c3 << 24);
}

template <bool BF16, bool ONESEG, bool ACT>
__global__ __launch_bounds__(256) void quantize_act_fast_kernel(const void* __restrict__ x, int8_t* __restrict__ xq,
                                                                uint32_t nchunks, uint32_t kchunks, uint32_t kmagic,
                                                                const ActTable tb) {
  constexpr int NL = BF16 ? 2 : 4;                       // 16-byte loads per chunk
  const uint32_t base = blockIdx.x * (256u * kActUnroll) + threadIdx.x;
  v4i raw[kActUnroll][NL];
#pragma unroll
  for (int j = 0; j < kActUnroll; ++j) {
    const uint32_t c = base + j * 256u;
    if (c < nchunks) {
      // x is read once and dead afterwards: non-temporal loads keep it from displacing X^ (which the GEMM reads
      // next) in the caches; 4.7 -> 5.2 TB/s.  The stores stay ordinary: non-temporal ones were slower.
#pragma unroll
      for (int l = 0; l < NL; ++l) raw[j][l] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(x) + ((size_t)NL * c + l));
    }
  }
#pragma unroll
  for (int j = 0; j < kActUnroll; ++j) {
    const uint32_t c = base + j * 256u;
    if (c >= nchunks) continue;
    float sp = tb.s_pos[0], sn = tb.s_neg[0], ip = tb.inv_pos[0], in = tb.inv_neg[0];
    bool dual = tb.dual[0] != 0;
    int acode = ACT ? tb.act[0] : SQ_ACT_NONE;
    if (!ONESEG) {
      // column of this chunk: c mod kchunks via a reciprocal multiply (q is exact or one too small)
      uint32_t q = __umulhi(c, kmagic);
      uint32_t r = c - q * kchunks;
      if (r >= kchunks) r -= kchunks;
      const int col = (int)(r * (uint32_t)kActChunk);
      for (int s = 1; s < tb.S; ++s) {
        if (col >= tb.kseg_off[s]) {
          sp = tb.s_pos[s]; sn = tb.s_neg[s]; ip = tb.inv_pos[s]; in = tb.inv_neg[s]; dual = tb.dual[s] != 0;
          if (ACT) acode = tb.act[s];
        }
      }
    }
    v4i out;
    auto values = [&](const int g, float (&v)[4]) __attribute__((always_inline)) {   // the four of output dword g
      if (BF16) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint32_t u = (uint32_t)raw[j][BF16 ? g / 2 : 0][(g % 2) * 2 + i];
          v[2 * i] = __uint_as_float(u << 16);
          v[2 * i + 1] = __uint_as_float(u & 0xFFFF0000u);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __int_as_float(raw[j][BF16 ? 0 : g][i]);
      }
    };
    if constexpr (!ACT) {
      // round_quotient()'s product for the four values of a dword, their distance from a tie tested once: clipped first (127 is no
      // tie), rounded by adding 1.5 * 2^23, whose low byte is then the code.  A NaN reciprocal always divides.  All waves of a few
      // rounds load, compute and store in step, so the instructions show: 64 x 256 fp32 3.1 -> 2.6 us, 8500 x 1536 bf16 9.7 -> 9.0
      // (least of 30).  One test for all sixteen values would send a fifth of the waves back.
      constexpr float kRound = 12582912.0f;
      const float divide = ip == ip && (!dual || in == in) ? 0.0f : 1.0f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float v[4], worst = divide;
        values(g, v);
        uint32_t u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float q = __builtin_fminf(__builtin_fmaxf(v[i] * (dual && v[i] < 0.0f ? in : ip), -kQmax), kQmax);
          const float r = q + kRound;
          worst = __builtin_fmaxf(worst, __builtin_fabsf(q - (r - kRound)));
          u[i] = __float_as_uint(r);
        }
        if (!(worst < kTieDistance)) {
#pragma unroll
          for (int i = 0; i < 4; ++i) u[i] = (uint32_t)clip_code(__builtin_rintf(v[i] / (dual && v[i] < 0.0f ? sn : sp)));
        }
        out[g] = (int)(__builtin_amdgcn_perm(u[1], u[0], 0x0C0C0400u) | __builtin_amdgcn_perm(u[3], u[2], 0x04000C0Cu));
      }
      reinterpret_cast<v4i*>(xq)[c] = out;
      continue;
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {                        // four output dwords of four codes
      float v[4];
      values(g, v);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = activate(acode, v[i]);
      int code[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ng = dual && (v[i] < 0.0f);          // X_- = min(X, 0) takes the s_- branch of Q_dual
        code[i] = clip_code(round_quotient(v[i], ng ? sn : sp, ng ? in : ip));
      }
      out[g] = (int)pack4(code[0], code[1], code[2], code[3]);
    }
    reinterpret_cast<v4i*>(xq)[c] = out;
  }
}

// Any K / segment alignment: one element per thread.
template <bool BF16, bool ACT>
__global__ __launch_bounds__(256) void quantize_act_generic_kernel(const void* __restrict__ x, int8_t* __restrict__ xq,
                                                                   int M, int K, const ActTable tb) {
  const size_t total = (size_t)M * K;
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < total; i += (size_t)gridDim.x * 256) {
    const int col = (int)(i % (size_t)K);
    float sp = tb.s_pos[0], sn = tb.s_neg[0], ip = tb.inv_pos[0], in = tb.inv_neg[0];
    bool dual = tb.dual[0] != 0;
    int acode = ACT ? tb.act[0] : SQ_ACT_NONE;
    for (int s = 1; s < tb.S; ++s) {
      if (col >= tb.kseg_off[s]) {
        sp = tb.s_pos[s]; sn = tb.s_neg[s]; ip = tb.inv_pos[s]; in = tb.inv_neg[s]; dual = tb.dual[s] != 0;
        if (ACT) acode = tb.act[s];
      }
    }
    float v = BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(x)[i]) : reinterpret_cast<const float*>(x)[i];
    if (ACT) v = activate(acode, v);
    const bool ng = dual && (v < 0.0f);
    xq[i] = (int8_t)clip_code(round_quotient(v, ng ? sn : sp, ng ? in : ip));
  }
}

template <bool ACT>
static hipError_t launch_quantize_act_impl(const void* x, bool x_is_bf16, int8_t* xq, int M, int K, const ActTable& tb,
                                           hipStream_t st) {
  bool aligned = (K % kActChunk == 0) && (reinterpret_cast<uintptr_t>(x) % 16 == 0) &&
                 (reinterpret_cast<uintptr_t>(xq) % 16 == 0);
  for (int s = 0; s <= tb.S; ++s) aligned = aligned && (tb.kseg_off[s] % kActChunk == 0);
  if (aligned) {
    const uint32_t kchunks = (uint32_t)(K / kActChunk);
    const uint32_t nchunks = (uint32_t)(((size_t)M * K) / kActChunk);
    const uint32_t kmagic = (uint32_t)(0x100000000ull / kchunks > 0xFFFFFFFFull ? 0xFFFFFFFFull : 0x100000000ull / kchunks);
    const unsigned blocks = (nchunks + 256u * kActUnroll - 1) / (256u * kActUnroll);
    const bool one = (tb.S == 1);
#define SQ_LAUNCH_ACT(B, O) \
  hipLaunchKernelGGL((quantize_act_fast_kernel<B, O, ACT>), dim3(blocks), dim3(256), 0, st, x, xq, nchunks, kchunks, kmagic, tb)
    if (x_is_bf16) { if (one) SQ_LAUNCH_ACT(true, true); else SQ_LAUNCH_ACT(true, false); }
    else           { if (one) SQ_LAUNCH_ACT(false, true); else SQ_LAUNCH_ACT(false, false); }
#undef SQ_LAUNCH_ACT
  } else {
    const size_t total = (size_t)M * K;
    const unsigned blocks = (unsigned)((total + 255) / 256 > 65536 ? 65536 : (total + 255) / 256);
    if (x_is_bf16) hipLaunchKernelGGL((quantize_act_generic_kernel<true, ACT>), dim3(blocks), dim3(256), 0, st, x, xq, M, K, tb);
    else           hipLaunchKernelGGL((quantize_act_generic_kernel<false, ACT>), dim3(blocks), dim3(256), 0, st, x, xq, M, K, tb);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Fused activation + quantizer for bf16 inputs by table.  A bf16 number has 65536 bit patterns, and the map
// h -> code of Q_dual(act(h)) of a K-segment is a byte per pattern.  Most of it is constant: below 2^lo with 2^lo at most half
// the smaller step (|act(x)| <= |x|: the quotient is below 1/2; fp8: 2^-10, half the smallest code) the code is 0.  So a workgroup
// fills the patterns of [2^lo, 2^5) of its segment, 14 - 22 binades of 256, with the very arithmetic of the direct path (the
// codes are the same to the bit), zeroes the rest, and then turns every element into one LDS byte read at the pattern
// itself; a chunk with a magnitude of 32 or more goes through the arithmetic.  HBM-bound: the direct path costs ~50 ALU
// instructions per element.  4608 x 15360 bf16, GELU on 12288 columns: 40.6 us in one launch (5.2 TB/s; 44 us with tables of
// all 65536 patterns, filled by a launch of their own into a workspace and copied to LDS; direct path 66 us); 2048 x 4608:
// 8.3 us (12.7).  One 1024-thread workgroup per compute unit; a second one, with a table of its own, changes nothing.
// ------------------------------------------------------------------------------------------------
constexpr int kTabThreads = 1024;
constexpr int kTabTop = (127 + 5) << 7;                  // first magnitude pattern beyond the table: 32.0
constexpr int kTabBytes = 0x8000 + kTabTop;              // indexed by the 16-bit pattern, both signs
constexpr int kTabUnit = 8192;                           // elements per compute unit for which a table of kTabBinades pays ...
constexpr int kTabBinades = 28;
constexpr int kTabMoreBinades = 12;                      // ... and what another kTabUnit pays for

struct TabPlan {
  int wg_begin[SQ_MAX_SEGMENTS + 1];                     // workgroups [wg_begin[s], wg_begin[s+1]) stream K-segment s
  int low[SQ_MAX_SEGMENTS];                              // first magnitude pattern with a code of its own
};

template <bool FP8>
__global__ __launch_bounds__(kTabThreads) void quantize_act_table_kernel(const uint16_t* __restrict__ h, int8_t* __restrict__ xq,
                                                                         int M, int K, const ActTable tb, const TabPlan plan) {
  __shared__ __attribute__((aligned(16))) uint8_t table[kTabBytes];
  int ks = 0;
  for (int s = 1; s < tb.S; ++s)
    if ((int)blockIdx.x >= plan.wg_begin[s]) ks = s;
  const int k0 = tb.kseg_off[ks], wg0 = plan.wg_begin[ks], wg1 = plan.wg_begin[ks + 1], low = plan.low[ks];
  const float sp = tb.s_pos[ks], sn = tb.s_neg[ks], ip = tb.inv_pos[ks], in = tb.inv_neg[ks];
  const bool dual = tb.dual[ks] != 0;
  const int acode = tb.act[ks];
  auto code_of = [&](const float x) __attribute__((always_inline)) -> uint32_t {
    const float v = activate(acode, x);
    const bool ng = dual && (v < 0.0f);
    if (FP8) return fp8_encode(v / (ng ? sn : sp));
    return (uint32_t)clip_code(round_quotient(v, ng ? sn : sp, ng ? in : ip)) & 0xFFu;
  };
  // chunk c of this workgroup's share of the segment: 16 elements of one row
  const uint32_t cps = (uint32_t)(tb.kseg_off[ks + 1] - k0) / kActChunk, nchunks = (uint32_t)M * cps;
  const uint32_t stride = (uint32_t)(wg1 - wg0) * kTabThreads, dr = stride / cps, dc = stride - dr * cps;
  uint32_t c = (uint32_t)((int)blockIdx.x - wg0) * kTabThreads + threadIdx.x, r = c / cps, cc = c - r * cps;
  v4i raw[2] = {(v4i)(0), (v4i)(0)};
  size_t at = 0;
  auto fetch = [&]() __attribute__((always_inline)) {    // x is read once and dead afterwards: non-temporal
    at = (size_t)r * K + k0 + (size_t)cc * kActChunk;
    const v4i* p = reinterpret_cast<const v4i*>(h + at);
    raw[0] = __builtin_nontemporal_load(p);
    raw[1] = __builtin_nontemporal_load(p + 1);
  };
  if (c < nchunks) fetch();                              // under the fill of the table
  for (int i = threadIdx.x; i < kTabBytes / 16; i += kTabThreads) reinterpret_cast<v4i*>(table)[i] = (v4i)(0);
  __syncthreads();
  for (int i = threadIdx.x; i < 2 * (kTabTop - low); i += kTabThreads) {
    const uint32_t bits = (uint32_t)(low + (i >> 1)) | ((i & 1) ? 0x8000u : 0u);
    table[bits] = (uint8_t)code_of(__uint_as_float(bits << 16));
  }
  __syncthreads();
  while (c < nchunks) {
    const v4i cur[2] = {raw[0], raw[1]};
    const size_t to = at;
    c += stride;
    r += dr;
    cc += dc;
    if (cc >= cps) { cc -= cps; ++r; }
    if (c < nchunks) fetch();
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    u16x2 top = {0, 0};
#pragma unroll
    for (int d = 0; d < 8; ++d) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, (uint32_t)cur[d >> 2][d & 3] & 0x7FFF7FFFu));
    v4i out;
    if (top[0] < kTabTop && top[1] < kTabTop) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t u0 = (uint32_t)cur[g / 2][(g % 2) * 2], u1 = (uint32_t)cur[g / 2][(g % 2) * 2 + 1];
        const uint32_t b0 = table[u0 & 0xFFFFu], b1 = table[u0 >> 16], b2 = table[u1 & 0xFFFFu], b3 = table[u1 >> 16];
        out[g] = (int)(b0 | (b1 << 8) | (b2 << 16) | (b3 << 24));
      }
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const uint32_t u0 = (uint32_t)cur[g / 2][(g % 2) * 2], u1 = (uint32_t)cur[g / 2][(g % 2) * 2 + 1];
        out[g] = (int)(code_of(__uint_as_float(u0 << 16)) | (code_of(__uint_as_float(u0 & 0xFFFF0000u)) << 8) |
                       (code_of(__uint_as_float(u1 << 16)) << 16) | (code_of(__uint_as_float(u1 & 0xFFFF0000u)) << 24));
      }
    }
    *reinterpret_cast<v4i*>(xq + to) = out;
  }
}

size_t quantize_act_fused_workspace_bytes(int S) { return (size_t)S * 65536; }

// The table kernel's launch, or false where the direct path serves: no activation, fp32 or unaligned input, or a matrix too small
// for the fill.  A binade of both signs costs a workgroup 0.08 - 0.1 us, an element 0.4 ns of a compute unit's time less than the
// direct path.  Table / direct in us, int8 and fp8: 348 x 6144 (8352 elements per compute unit), 13 - 27 binades 5.5 - 6.8 / 6.1 -
// 6.6, 46 binades 8.6 / 6.4; 683 x 6144, 33 binades 7.5 / 8.3, 47 binades 8.9 / 8.4; 2048 x 4608, 65 binades 12.9 / 13.4, 125
// binades 18.9 / 13.4 (fp8 steps of 2^-50, 2^-110); 4608 x 15360, 29 binades 41.3 / 73.1 (fp8 step 2^-14).
bool launch_quantize_act_table(const void* h, bool h_is_bf16, int8_t* xq, int M, int K, const ActTable& tb, int cus, hipStream_t st,
                               bool fp8) {
  bool ok = h_is_bf16 && (K % kActChunk == 0) && (reinterpret_cast<uintptr_t>(h) % 16 == 0) &&
            (reinterpret_cast<uintptr_t>(xq) % 16 == 0) && (long long)M * K >= (long long)kTabUnit * cus;
  const long long more = (long long)kTabMoreBinades * M * K / ((long long)kTabUnit * cus) - kTabMoreBinades;
  const int lowest = more > 126 ? -126 : 5 - kTabBinades - (int)more < -126 ? -126 : 5 - kTabBinades - (int)more;
  bool any = false;
  TabPlan plan;
  const int total = cus > tb.S ? cus : tb.S;             // dealt to the K-segments in proportion to their width, one at least
  plan.wg_begin[0] = 0;
  for (int s = 0; s < tb.S; ++s) {
    ok = ok && tb.kseg_off[s] % kActChunk == 0;
    any = any || tb.act[s] != SQ_ACT_NONE;
    const float step = tb.dual[s] && tb.s_neg[s] < tb.s_pos[s] ? tb.s_neg[s] : tb.s_pos[s];
    int e = 0;
    (void)std::frexp(step, &e);                          // step in [2^(e-1), 2^e)
    const int lo = e - 1 - (fp8 ? 10 : 1);               // 2^lo <= step / 2 (fp8: step / 2^10)
    if (lo < lowest || lo > 4) ok = false;
    plan.low[s] = (127 + lo) << 7;
    plan.wg_begin[s + 1] = plan.wg_begin[s] + 1 + (int)((long long)(total - tb.S) * (tb.kseg_off[s + 1] - tb.kseg_off[s]) / K);
  }
  if (!ok || !any) return false;
  const dim3 grid(plan.wg_begin[tb.S]);
  const uint16_t* src = reinterpret_cast<const uint16_t*>(h);
  if (fp8) hipLaunchKernelGGL(quantize_act_table_kernel<true>, grid, dim3(kTabThreads), 0, st, src, xq, M, K, tb, plan);
  else hipLaunchKernelGGL(quantize_act_table_kernel<false>, grid, dim3(kTabThreads), 0, st, src, xq, M, K, tb, plan);
  return true;
}

// tb.act is read only when some K-segment has an activation fused in front of it (sq_quantize_act_fused)
hipError_t launch_quantize_act(const void* x, bool x_is_bf16, int8_t* xq, int M, int K, const ActTable& tb,
                               hipStream_t st) {
  bool any = false;
  for (int s = 0; s < tb.S; ++s) any = any || tb.act[s] != SQ_ACT_NONE;
  if (any && launch_quantize_act_table(x, x_is_bf16, xq, M, K, tb, device_cus(), st, false)) return hipGetLastError();
  return any ? launch_quantize_act_impl<true>(x, x_is_bf16, xq, M, K, tb, st)
             : launch_quantize_act_impl<false>(x, x_is_bf16, xq, M, K, tb, st);
}

// ------------------------------------------------------------------------------------------------
// Weight quantize: one wavefront per (output channel n, K-segment ks).  Pass 1 reduces max |w| over the
// row segment, pass 2 re-reads it (L2-resident: a row segment is at most 0.5 MB) and writes the codes.
// ------------------------------------------------------------------------------------------------
template <bool BF16>
__device__ __forceinline__ float load_w(const void* w, size_t i) {
  return BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(w)[i]) : reinterpret_cast<const float*>(w)[i];
}

// MODE 0: per output channel and K-segment, both passes fused.  MODE 1: first pass only, the row maximum goes to
// wscale[ks][n].  MODE 2: second pass only, with the step found in wscale[ks][n] (block-granular quantizer).
template <bool BF16, bool VEC4, int MODE>
__global__ __launch_bounds__(256) void quantize_weight_kernel(const void* __restrict__ w, int8_t* __restrict__ wq,
                                                              float* __restrict__ wscale, int N, int K,
                                                              const KsegTable tb) {
  const int lane = threadIdx.x & 63;
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= (long)N * tb.S) return;            // whole wave leaves together
  const int n = (int)(item / tb.S), ks = (int)(item % tb.S);
  int k0 = 0, k1 = 0;
  for (int s = 0; s < tb.S; ++s)
    if (s == ks) { k0 = tb.off[s]; k1 = tb.off[s + 1]; }
  const size_t row = (size_t)n * K;
  float sw;
  if (MODE == 2) {
    sw = wscale[(size_t)ks * N + n];
  } else {
    float a = 0.0f;
    if (VEC4) {
      for (int k = k0 + 4 * lane; k < k1; k += 256) {
#pragma unroll
        for (int i = 0; i < 4; ++i) a = __builtin_fmaxf(a, __builtin_fabsf(load_w<BF16>(w, row + k + i)));
      }
    } else {
      for (int k = k0 + lane; k < k1; k += 64) a = __builtin_fmaxf(a, __builtin_fabsf(load_w<BF16>(w, row + k)));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) a = __builtin_fmaxf(a, __shfl_xor(a, off, 64));
    if (MODE == 1) {
      if (lane == 0) wscale[(size_t)ks * N + n] = a;
      return;
    }
    sw = (a == 0.0f) ? 1.0f : a / kQmax;
    if (lane == 0) wscale[(size_t)ks * N + n] = sw;
  }
  if (VEC4) {
    for (int k = k0 + 4 * lane; k < k1; k += 256) {
      int c[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i] = clip_code(__builtin_rintf(load_w<BF16>(w, row + k + i) / sw));
      *reinterpret_cast<uint32_t*>(wq + row + k) = pack4(c[0], c[1], c[2], c[3]);
    }
  } else {
    for (int k = k0 + lane; k < k1; k += 64) wq[row + k] = (int8_t)clip_code(__builtin_rintf(load_w<BF16>(w, row + k) / sw));
  }
}

template <int MODE>
static void launch_weight_pass(const void* w, bool w_is_bf16, int8_t* wq, float* wscale, int N, int K, const KsegTable& tb,
                               hipStream_t st) {
  bool vec = (K % 4 == 0) && (reinterpret_cast<uintptr_t>(w) % 16 == 0) && (reinterpret_cast<uintptr_t>(wq) % 4 == 0);
  for (int s = 0; s <= tb.S; ++s) vec = vec && (tb.off[s] % 4 == 0);
  const long items = (long)N * tb.S;
  const unsigned blocks = (unsigned)((items + 3) / 4);
#define SQ_LAUNCH_W(B, V) hipLaunchKernelGGL((quantize_weight_kernel<B, V, MODE>), dim3(blocks), dim3(256), 0, st, w, wq, wscale, N, K, tb)
  if (w_is_bf16) { if (vec) SQ_LAUNCH_W(true, true); else SQ_LAUNCH_W(true, false); }
  else           { if (vec) SQ_LAUNCH_W(false, true); else SQ_LAUNCH_W(false, false); }
#undef SQ_LAUNCH_W
}

// ------------------------------------------------------------------------------------------------
// Weight quantize of aligned rows (8-bit codes, or 4-bit codes in the packed order of quantize_weight_w4_kernel): TPI threads
// own one (output channel, K-segment) and keep it in registers between the maximum and the codes, so W is read once, by up
// to NCH independent 16-byte loads per thread.  The code is round_quotient()'s, bit-identical to the division (one in a few
// thousand elements divides).  HBM-bound: 3072 x 15360 fp32, two K-segments (189 MB in): 8 bit 44 us (5.3 TB/s), 4 bit 42
// (5.0 TB/s), against 83 and 108 of the one-wave-per-row kernels that read the row twice and divide every element.  A workgroup
// is short, so the chain in front of its loads counts: the grid's second dimension is the K-segment (no division, the segment's
// bounds by scalar loads), and loads beyond the segment repeat its last elements where a test on each kept two of them apart
// from the rest and put a wait between them (8 bit 50, 4 bit 45 us; 4096 x 20480 83 -> 75, bf16 3072 x 15360 38 -> 30).
// ------------------------------------------------------------------------------------------------
template <bool BF16, int BITS, int TPI, int NCH>
__global__ __launch_bounds__(256) void quantize_weight_row_kernel(const void* __restrict__ w, uint8_t* __restrict__ out,
                                                                  float* __restrict__ wscale, int N, int K, const KsegTable tb) {
  constexpr int CE = BF16 ? 8 : 4;                 // elements of a 16-byte load
  constexpr int PS = 64 / CE;                      // 4 bit: pairs of loads (64 columns apart) per 128-code step
  const int rows = BITS == 4 ? (N + 15) & ~15 : N;
  const int t = threadIdx.x % TPI;
  unsigned block = blockIdx.x;
  // 4 bit, wide fp32 rows: the 16 rows that share the packed lines go to one XCD (workgroup ids go round the eight; 3072 x 15360 43.6
  // -> 42.2 us, 4096 x 20480 73.4 -> 70.8; 12288 x 3072 31.0 / 31.9, bf16 2048 x 10240 15.4 / 15.8)
  if (BITS == 4 && !BF16 && NCH >= 8) {
    constexpr unsigned G = 16 * TPI / 256;         // workgroups of such a group
    if (block < gridDim.x / (8 * G) * (8 * G)) block = block / (8 * G) * (8 * G) + block % 8 * G + block / 8 % G;
  }
  // 4 bit, long fp32 rows: from the last row to the first.  Both formats are often made of one weight, the 8-bit codes first, and the end
  // of it may still be in the Infinity Cache (3072 x 15360, both behind the two calibrations of 4608 rows 153.1 -> 150.2 us; shorter
  // rows gained nothing.  The 8-bit pass reading through that cache: 149, but 47 instead of 44 us by itself).
  constexpr bool BACK = BITS == 4 && !BF16 && NCH >= 16;
  if (BACK) block = gridDim.x - 1 - block;
  const int n = block * (256 / TPI) + __builtin_amdgcn_readfirstlane(threadIdx.x / TPI);
  const int ks = BACK ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  if (n >= rows) return;                           // a whole wave (TPI 64) or workgroup leaves together
  const int k0 = tb.off[ks], L = tb.off[ks + 1] - k0;
  auto column = [&](const int l) __attribute__((always_inline)) {   // first column, inside the segment, of load l
    if (BITS == 8) return (t + TPI * l) * CE;
    const int p = t + TPI * (l >> 1);
    return (p / PS) * 128 + (p % PS) * CE + 64 * (l & 1);
  };
  auto packed_at = [&](const int l) __attribute__((always_inline)) {   // 4 bit: where the codes of loads l, l + 1 go
    const int p = t + TPI * (l >> 1);
    return out + (((size_t)(n >> 4) * (K >> 7) + (k0 >> 7) + p / PS) * 16 + (n & 15)) * 64 + (p % PS) * CE;
  };
  auto store = [](uint8_t* to, const uint32_t lo, const uint32_t hi) __attribute__((always_inline)) {
    if (BF16) *reinterpret_cast<uint2*>(to) = make_uint2(lo, hi);
    else *reinterpret_cast<uint32_t*>(to) = lo;
  };
  if (BITS == 4 && n >= N) {                       // padding row of the last group of 16
#pragma unroll
    for (int l = 0; l < NCH; l += 2)
      if (column(l) < L) store(packed_at(l), 0u, 0u);
    return;
  }
  const size_t row = (size_t)n * K + k0;
  v4i raw[NCH];
#pragma unroll
  for (int l = 0; l < NCH; ++l) {                  // beyond the segment: its last elements again, which no maximum minds
    const int c = column(l) < L ? column(l) : L - CE;
    raw[l] = BF16 ? __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(w) + row + c))
                  : __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const float*>(w) + row + c));
  }
  auto value = [&](const int l, const int i) __attribute__((always_inline)) {
    if (!BF16) return __int_as_float(raw[l][i & 3]);
    const uint32_t u = (uint32_t)raw[l][i >> 1];
    return __uint_as_float((i & 1) ? (u & 0xFFFF0000u) : (u << 16));
  };
  float a = 0.0f;
#pragma unroll
  for (int l = 0; l < NCH; ++l)
#pragma unroll
    for (int i = 0; i < CE; ++i) a = __builtin_fmaxf(a, __builtin_fabsf(value(l, i)));
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) a = __builtin_fmaxf(a, __shfl_xor(a, off, 64));
  if (TPI == 256) {
    __shared__ float red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    a = __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
  }
  constexpr float QM = BITS == 8 ? kQmax : 7.0f;
  const float sw = (a == 0.0f) ? 1.0f : a / QM;
  const float inv = (sw >= 1e-30f && sw <= 1e30f) ? 1.0f / sw : __builtin_nanf("");
  if (t == 0) wscale[(size_t)ks * N + n] = sw;
  auto code = [&](const int l, const int i) __attribute__((always_inline)) {
    return (int)__builtin_fminf(__builtin_fmaxf(round_quotient(value(l, i), sw, inv), -QM), QM);
  };
#pragma unroll
  for (int l = 0; l < NCH; l += BITS == 8 ? 1 : 2) {
    if (column(l) >= L) continue;
    uint32_t pk[2] = {0u, 0u};
    if (BITS == 8) {
#pragma unroll
      for (int i = 0; i < CE; ++i) pk[i >> 2] |= (uint32_t)(code(l, i) & 0xFF) << (8 * (i & 3));
      store(out + row + column(l), pk[0], pk[1]);
    } else {
#pragma unroll
      for (int i = 0; i < CE; ++i)
        pk[i >> 2] |= (uint32_t)((code(l, i) & 0xF) | ((code(l + 1 < NCH ? l + 1 : l, i) & 0xF) << 4)) << (8 * (i & 3));
      store(packed_at(l), pk[0], pk[1]);
    }
  }
}

// Threads and loads per row segment by the longest segment: a wave for up to 2048 fp32 (4096 bf16) columns, a workgroup beyond
// 1024 (2048) where there are too few segments to give every compute unit eight waves, and always beyond 2048 (4096); longer
// rows than a workgroup's registers hold (16384 / 32768 columns) and unaligned ones keep the two-read kernels.  So do short
// segments that leave most of a wave without work (to the left this kernel, to the right the two-read one: bf16 13824 rows of
// 256, 8 bit 7.8 / 6.8 us, 384, 4 bit 10.1 / 9.2, 512, 4 bit 10.6 / 11.7; fp32 13824 rows of 128, 4 bit 7.1 / 6.6).  A wave
// against a workgroup: fp32 6912 x 1152, 8 bit 8.6 / 12.5 us (two-read 10.7), 384 x 1152 4.1 / 3.8.  One long segment among
// many short ones, each of which would get as many threads, goes there too (fp32 3072 x 3200, 2176 columns and eight times 128,
// 8 bit 31.0 / 19.8; 1024 x 16384, 16000 columns and three times 128, 42 / 46).
template <int BITS>
static bool launch_weight_rows(const void* w, bool w_is_bf16, uint8_t* out, float* wscale, int N, int K, const KsegTable& tb,
                               hipStream_t st) {
  const int ce = w_is_bf16 ? 8 : 4;
  int longest = 0;
  bool ok = K % ce == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0 && reinterpret_cast<uintptr_t>(out) % 8 == 0;
  for (int s = 0; s < tb.S; ++s) {
    const int L = tb.off[s + 1] - tb.off[s];
    longest = L > longest ? L : longest;
    ok = ok && tb.off[s] % ce == 0;
  }
  const int shortest = w_is_bf16 ? (BITS == 8 ? 257 : 385) : (BITS == 8 ? 1 : 129);
  if (!ok || longest > 256 * 16 * ce || longest < shortest) return false;
  if (longest > 64 * 4 * ce && (BITS == 8 ? 4ll : 6ll) * K < (long long)tb.S * longest) return false;
  const int rows = BITS == 4 ? (N + 15) & ~15 : N;
  const long items = (long)rows * tb.S;
#define SQ_ROWS(B, T, C) hipLaunchKernelGGL((quantize_weight_row_kernel<B, BITS, T, C>), dim3((unsigned)((rows + 256 / T - 1) / (256 / T)), tb.S), dim3(256), 0, st, w, out, wscale, N, K, tb)
#define SQ_PICK(B) \
  if (longest <= 64 * 4 * ce) SQ_ROWS(B, 64, 4); \
  else if (longest <= 64 * 8 * ce && items >= 2048) SQ_ROWS(B, 64, 8); \
  else if (longest <= 256 * 4 * ce) SQ_ROWS(B, 256, 4); \
  else if (longest <= 256 * 8 * ce) SQ_ROWS(B, 256, 8); \
  else SQ_ROWS(B, 256, 16)
  if (w_is_bf16) { SQ_PICK(true); }
  else           { SQ_PICK(false); }
#undef SQ_PICK
#undef SQ_ROWS
  return true;
}

hipError_t launch_quantize_weight(const void* w, bool w_is_bf16, int8_t* wq, float* wscale, int N, int K,
                                  const KsegTable& tb, hipStream_t st) {
  if (!launch_weight_rows<8>(w, w_is_bf16, reinterpret_cast<uint8_t*>(wq), wscale, N, K, tb, st))
    launch_weight_pass<0>(w, w_is_bf16, wq, wscale, N, K, tb, st);
  return hipGetLastError();
}

// Block-granular steps: wscale[ks][n] holds the row maxima on entry; one workgroup per (K-segment, N-segment) block
// reduces them and writes the block's step back to every channel of the block.
__global__ __launch_bounds__(256) void weight_block_step_kernel(float* __restrict__ wscale, int N, const KsegTable nt) {
  const int ks = blockIdx.y, ns = blockIdx.x;
  int n0 = 0, n1 = 0;
  for (int t = 0; t < nt.S; ++t)
    if (t == ns) { n0 = nt.off[t]; n1 = nt.off[t + 1]; }
  float* row = wscale + (size_t)ks * N;
  float a = 0.0f;
  for (int n = n0 + threadIdx.x; n < n1; n += 256) a = __builtin_fmaxf(a, row[n]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) a = __builtin_fmaxf(a, __shfl_xor(a, off, 64));
  __shared__ float red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  a = __builtin_fmaxf(__builtin_fmaxf(red[0], red[1]), __builtin_fmaxf(red[2], red[3]));
  const float sw = (a == 0.0f) ? 1.0f : a / kQmax;
  __syncthreads();                                       // every thread has read the maxima before they are overwritten
  for (int n = n0 + threadIdx.x; n < n1; n += 256) row[n] = sw;
}

// One step per (K-segment, N-segment) block: row maxima, block reduce + broadcast, quantize with the block's step.
hipError_t launch_quantize_weight_block(const void* w, bool w_is_bf16, int8_t* wq, float* wscale, int N, int K,
                                        const KsegTable& kt, const KsegTable& nt, hipStream_t st) {
  launch_weight_pass<1>(w, w_is_bf16, wq, wscale, N, K, kt, st);
  hipLaunchKernelGGL(weight_block_step_kernel, dim3(nt.S, kt.S), dim3(256), 0, st, wscale, N, nt);
  launch_weight_pass<2>(w, w_is_bf16, wq, wscale, N, K, kt, st);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Dynamic per-token activation steps (App. B: in the 4-bit settings activations are quantized dynamically per
// token): one workgroup per token row; per K-segment the row's extremes give its steps by the min/max rule
// (Sec. 4.3.2: s_+ = max x / 127, s_- = |min x| / 127, 1.0 where the extreme is 0), then the row is quantized with
// them.  This kernel takes any shape; a row is read twice (the second time from cache).  tok_steps: [2][M][S], s_pos
// then s_neg.
// ------------------------------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void quantize_act_dynamic_kernel(const void* __restrict__ x, int8_t* __restrict__ xq,
                                                                   float* __restrict__ tok_steps, int M, int K,
                                                                   const ActTable tb, const float qmax) {
  const int m = blockIdx.x;
  const size_t row = (size_t)m * K;
  __shared__ float red[2][4];
  __shared__ float stp[2];
  for (int ks = 0; ks < tb.S; ++ks) {
    const int k0 = tb.kseg_off[ks], k1 = tb.kseg_off[ks + 1];
    const bool dual = tb.dual[ks] != 0;
    float mp = 0.0f, mn = 0.0f;
    for (int k = k0 + threadIdx.x; k < k1; k += 256) {
      const float v = load_w<BF16>(x, row + k);
      if (dual) {
        mp = __builtin_fmaxf(mp, v);
        mn = __builtin_fmaxf(mn, -v);
      } else {
        mp = __builtin_fmaxf(mp, __builtin_fabsf(v));
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      mp = __builtin_fmaxf(mp, __shfl_xor(mp, off, 64));
      mn = __builtin_fmaxf(mn, __shfl_xor(mn, off, 64));
    }
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = mp; red[1][threadIdx.x >> 6] = mn; }
    __syncthreads();
    if (threadIdx.x == 0) {
      mp = __builtin_fmaxf(__builtin_fmaxf(red[0][0], red[0][1]), __builtin_fmaxf(red[0][2], red[0][3]));
      mn = __builtin_fmaxf(__builtin_fmaxf(red[1][0], red[1][1]), __builtin_fmaxf(red[1][2], red[1][3]));
      const float sp = (mp == 0.0f) ? 1.0f : mp / qmax, sn = (mn == 0.0f) ? 1.0f : mn / qmax;
      stp[0] = sp;
      stp[1] = sn;
      tok_steps[(size_t)m * tb.S + ks] = sp;
      tok_steps[((size_t)M + m) * tb.S + ks] = sn;
    }
    __syncthreads();
    const float sp = stp[0], sn = stp[1];
    for (int k = k0 + threadIdx.x; k < k1; k += 256) {
      const float v = load_w<BF16>(x, row + k);
      const bool ng = dual && (v < 0.0f);
      xq[row + k] = (int8_t)clip_code(__builtin_rintf(v / (ng ? sn : sp)));
    }
    __syncthreads();                                      // stp and red are reused by the next segment
  }
}

// The same for aligned rows (K, the K-segment boundaries multiples of 16, 16-byte aligned pointers) of at most NCH chunks of G
// 16-byte loads per thread: TPR threads own a row and keep it in registers between the two passes, so the row is read once
// (at large M the rows in flight on an XCD exceed its L2 and a second read goes back to memory), the loads are streaming and
// the quotient is the reciprocal product of round_quotient (bit-identical to the division).  G: 1, or a chunk of 16 elements, whose
// segment tests, step reads and store are shared by its loads.
template <bool BF16, int TPR, int NCH, int G>
__global__ __launch_bounds__(256) void quantize_act_dynamic_fast_kernel(const void* __restrict__ x, int8_t* __restrict__ xq,
                                                                        float* __restrict__ tok_steps, int M, int K,
                                                                        const ActTable tb, const float qmax) {
  constexpr int CE = BF16 ? 8 : 4;                       // elements of a 16-byte load
  constexpr int CC = G * CE;                             // elements of a chunk
  constexpr int RPW = 256 / TPR;                         // rows of the workgroup
  static_assert(CC <= 16, "K and the boundaries are multiples of 16 only");
  const int t = threadIdx.x % TPR, wrow = threadIdx.x / TPR;
  const int mr = blockIdx.x * RPW + wrow;
  const int m = mr < M ? mr : M - 1;                     // rows beyond M do the last one again: same values, same places
  const size_t row = (size_t)m * K;
  __shared__ float red[2][4];
  __shared__ float stp[RPW][SQ_MAX_SEGMENTS][4];         // s_+, s_-, and their reciprocals (NaN: always divide)
  v4i raw[NCH][G];
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int col = (t + TPR * j) * CC;
#pragma unroll
    for (int l = 0; l < G; ++l) raw[j][l] = (v4i)(0);
    if (col < K) {
#pragma unroll
      for (int l = 0; l < G; ++l)
        raw[j][l] = BF16 ? __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(x) + row + col) + l)
                         : __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const float*>(x) + row + col) + l);
    }
  }
  auto value = [&](const int j, const int e) __attribute__((always_inline)) -> float {   // element e of chunk j (constants)
    if (!BF16) return __int_as_float(raw[j][(e >> 2) % G][e & 3]);
    const uint32_t u = (uint32_t)raw[j][(e >> 3) % G][(e >> 1) & 3];
    return __uint_as_float((e & 1) ? (u & 0xFFFF0000u) : (u << 16));
  };
  for (int ks = 0; ks < tb.S; ++ks) {
    const int k0 = tb.kseg_off[ks], k1 = tb.kseg_off[ks + 1];
    const bool dual = tb.dual[ks] != 0;
    float mp = 0.0f, mn = 0.0f;
    if (BF16) {
      // Extremes on the bit patterns, two elements per instruction: as signed 16-bit integers the positive bf16 numbers
      // keep their order and every negative one is below zero (max with 0 = pattern of max(x, 0)); as unsigned ones the
      // negative numbers lie above all positive ones, ordered by magnitude (a maximum >= 0x8000 is the pattern of min x).
      typedef short s16x2 __attribute__((ext_vector_type(2)));
      typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
      s16x2 hi_s = {0, 0};
      u16x2 hi_u = {0, 0};
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        const int col = (t + TPR * j) * CC;
        if (col < K && col >= k0 && col < k1) {
#pragma unroll
          for (int d = 0; d < 4 * G; ++d) {
            const int w = raw[j][d / 4][d % 4];
            if (dual) {
              hi_s = __builtin_elementwise_max(hi_s, __builtin_bit_cast(s16x2, w));
              hi_u = __builtin_elementwise_max(hi_u, __builtin_bit_cast(u16x2, w));
            } else {
              hi_u = __builtin_elementwise_max(hi_u, __builtin_bit_cast(u16x2, w & 0x7FFF7FFF));
            }
          }
        }
      }
      const uint32_t us = (uint32_t)(hi_s[0] > hi_s[1] ? hi_s[0] : hi_s[1]);
      const uint32_t uu = (uint32_t)(hi_u[0] > hi_u[1] ? hi_u[0] : hi_u[1]);
      if (dual) {
        mp = __uint_as_float(us << 16);
        mn = uu >= 0x8000u ? __uint_as_float((uu & 0x7FFFu) << 16) : 0.0f;
      } else {
        mp = __uint_as_float(uu << 16);
      }
    } else {
#pragma unroll
      for (int j = 0; j < NCH; ++j) {
        const int col = (t + TPR * j) * CC;
        if (col < K && col >= k0 && col < k1) {
#pragma unroll
          for (int e = 0; e < CC; ++e) {
            const float v = value(j, e);
            if (dual) {
              mp = __builtin_fmaxf(mp, v);
              mn = __builtin_fmaxf(mn, -v);
            } else {
              mp = __builtin_fmaxf(mp, __builtin_fabsf(v));
            }
          }
        }
      }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      mp = __builtin_fmaxf(mp, __shfl_xor(mp, off, 64));
      mn = __builtin_fmaxf(mn, __shfl_xor(mn, off, 64));
    }
    if (TPR > 64) {
      if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = mp; red[1][threadIdx.x >> 6] = mn; }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < TPR / 64; ++i) {
        mp = __builtin_fmaxf(mp, red[0][wrow * (TPR / 64) + i]);
        mn = __builtin_fmaxf(mn, red[1][wrow * (TPR / 64) + i]);
      }
    }
    if (t == 0) {
      const float sp = (mp == 0.0f) ? 1.0f : mp / qmax, sn = (mn == 0.0f) ? 1.0f : mn / qmax;
      stp[wrow][ks][0] = sp;
      stp[wrow][ks][1] = sn;
      stp[wrow][ks][2] = (sp >= 1e-30f && sp <= 1e30f) ? 1.0f / sp : __builtin_nanf("");
      stp[wrow][ks][3] = (sn >= 1e-30f && sn <= 1e30f) ? 1.0f / sn : __builtin_nanf("");
      tok_steps[(size_t)m * tb.S + ks] = sp;
      tok_steps[((size_t)M + m) * tb.S + ks] = sn;
    }
    if (TPR > 64) __syncthreads();                        // red is reused by the next segment; stp is complete after the last
#pragma unroll
    for (int j = 0; j < NCH; ++j)
#pragma unroll
      for (int l = 0; l < G; ++l) asm volatile("" : "+v"(raw[j][l]));   // keep the row as loaded: widened copies held across the
  }                                                                     // passes would cost half the occupancy
  if (TPR == 64) {                                        // lane 0's steps, to this wave's other lanes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int col = (t + TPR * j) * CC;
    if (col >= K) continue;
    int ks = 0;
    bool dual = tb.dual[0] != 0;
    for (int sg = 1; sg < tb.S; ++sg)
      if (col >= tb.kseg_off[sg]) { ks = sg; dual = tb.dual[sg] != 0; }
    const float sp = stp[wrow][ks][0], sn = stp[wrow][ks][1], ip = stp[wrow][ks][2], in = stp[wrow][ks][3];
    int out[4];
#pragma unroll
    for (int q = 0; q < CC / 4; ++q) {
      int code[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = value(j, 4 * q + i);
        const bool ng = dual && (v < 0.0f);
        code[i] = clip_code(round_quotient(v, ng ? sn : sp, ng ? in : ip));
      }
      out[q] = (int)pack4(code[0], code[1], code[2], code[3]);
    }
    if (CC == 16) *reinterpret_cast<v4i*>(xq + row + col) = (v4i){out[0], out[1], out[2], out[3]};
    else if (CC == 8) *reinterpret_cast<v2i*>(xq + row + col) = (v2i){out[0], out[1]};
    else *reinterpret_cast<int*>(xq + row + col) = out[0];
  }
}

hipError_t launch_quantize_act_dynamic(const void* x, bool x_is_bf16, int8_t* xq, float* tok_steps, int M, int K,
                                       const ActTable& tb, float qmax, hipStream_t st) {
  bool fast = K % 16 == 0 && K <= 4096 * 8 && (reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(xq)) % 16 == 0;
  for (int s = 0; s <= tb.S; ++s) fast = fast && tb.kseg_off[s] % 16 == 0;
  if (fast) {
    // Threads per row: a workgroup and the fewest loads per thread that hold the row, except where that leaves a quarter of the
    // threads or more without work and there are rows enough: up to 192 loads on a wave (8500 x 1536 bf16: 18.3 -> 13.6 us,
    // fp32 on half a workgroup 22.3 -> 16.9), 257 - 384 on half a workgroup (4096 x 3072 bf16, two K-segments: 15.4 -> 14.2).
    // Wider rows on fewer threads are slower (4096 x 4096 on a wave 18.5 us, on a workgroup 15.2), few rows are a matter
    // of latency (a workgroup each and a wave each: 16 x 1152 3.1 and 4.6 us, 1024 x 1536 4.4 and 5.8, 1500 x 1024 4.8 and 4.8,
    // 2048 x 512 4.9 and 4.1).
    const int loads = K / (x_is_bf16 ? 8 : 4);
    // Chunks of 16 elements instead of single loads: a workgroup's chunks fit such a row as well (up to 4096 columns and the
    // lengths beyond 6144; between them a second, nearly empty chunk per thread), and with about a row per compute unit or fewer the work
    // on each load shows (fp32 16 x 12288: 7.6 us, by single loads 9.7; 64 x 4096 4.6 and 5.1), as it does for the lengths that
    // one chunk per thread covers (bf16 2048 x 4096 8.4 and 8.8) and where 32 single loads cost the occupancy (fp32 4096 x 30720
    // 181 and 198).
    const bool chunks = K > 2048 && ((M <= device_cus() * 5 / 4 && (K <= 4096 || K > 6144)) || (x_is_bf16 ? K > 3072 && K <= 4096 : K > 16384));
#define SQ_D(B, T, N, G) hipLaunchKernelGGL((quantize_act_dynamic_fast_kernel<B, T, N, G>), dim3((M + 256 / T - 1) / (256 / T)), dim3(256), 0, st, x, xq, tok_steps, M, K, tb, qmax)
#define SQ_DN(B) do { \
    constexpr int C16 = B ? 2 : 4; \
    if (chunks) { \
      if (K <= 4096) SQ_D(B, 256, 1, C16); else if (K <= 8192) SQ_D(B, 256, 2, C16); else if (K <= 16384) SQ_D(B, 256, 4, C16); \
      else SQ_D(B, 256, 8, C16); \
    } else if (M >= (loads <= 64 ? 1024 : loads <= 128 ? 1536 : 2048) && loads <= 192) SQ_D(B, 64, 3, 1); \
    else if (M >= 2048 && loads > 256 && loads <= 384) SQ_D(B, 128, 3, 1); \
    else if (loads <= 256) SQ_D(B, 256, 1, 1); else if (loads <= 512) SQ_D(B, 256, 2, 1); else if (loads <= 768) SQ_D(B, 256, 3, 1); \
    else if (loads <= 1024) SQ_D(B, 256, 4, 1); else if (loads <= 1536) SQ_D(B, 256, 6, 1); else if (loads <= 2048) SQ_D(B, 256, 8, 1); \
    else SQ_D(B, 256, 16, 1); } while (0)
    if (x_is_bf16) SQ_DN(true); else SQ_DN(false);
#undef SQ_DN
#undef SQ_D
    return hipGetLastError();
  }
  if (x_is_bf16) hipLaunchKernelGGL((quantize_act_dynamic_kernel<true>), dim3(M), dim3(256), 0, st, x, xq, tok_steps, M, K, tb, qmax);
  else           hipLaunchKernelGGL((quantize_act_dynamic_kernel<false>), dim3(M), dim3(256), 0, st, x, xq, tok_steps, M, K, tb, qmax);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// GEGLU in front of the quantizer (App. B lists GEGLU with SiLU and GELU): h [M][2K] = [value | gate],
// xq[m][k] = Q_dual(value[m][k] * GELU(gate[m][k])) with the bit-specified GELU of activate() and one fp32 product.
// VEC: a thread owns 16 consecutive outputs (K, the K-segment boundaries multiples of 16, pointers 16-byte aligned);
// otherwise one output per thread.  HBM-bound where the gate's arithmetic lets it: 2 x 2 (bf16) or 2 x 4 bytes in,
// 1 byte out per element.
// ------------------------------------------------------------------------------------------------
template <bool BF16, bool VEC>
__global__ __launch_bounds__(256) void quantize_act_geglu_kernel(const void* __restrict__ h, int8_t* __restrict__ xq,
                                                                 int M, int K, const ActTable tb) {
#pragma clang fp contract(off)
  constexpr int W = VEC ? 16 : 1;
  const size_t nitem = (size_t)M * (size_t)(K / W);
  const int per_row = K / W;
  for (size_t c = blockIdx.x * (size_t)256 + threadIdx.x; c < nitem; c += (size_t)gridDim.x * 256) {
    const size_t m = c / per_row;
    const int col = (int)(c - m * per_row) * W;
    float sp = tb.s_pos[0], sn = tb.s_neg[0], ip = tb.inv_pos[0], in = tb.inv_neg[0];
    bool dual = tb.dual[0] != 0;
    for (int s = 1; s < tb.S; ++s) {
      if (col >= tb.kseg_off[s]) {
        sp = tb.s_pos[s]; sn = tb.s_neg[s]; ip = tb.inv_pos[s]; in = tb.inv_neg[s]; dual = tb.dual[s] != 0;
      }
    }
    const size_t ev = m * 2 * (size_t)K + col, eg = ev + K;       // value and gate of the first output
    float v[W], g[W];
    if (VEC) {
      if (BF16) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const v4i rv = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(h) + ev + 8 * q));
          const v4i rg = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(h) + eg + 8 * q));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[8 * q + 2 * i] = __uint_as_float((uint32_t)rv[i] << 16);
            v[8 * q + 2 * i + 1] = __uint_as_float((uint32_t)rv[i] & 0xFFFF0000u);
            g[8 * q + 2 * i] = __uint_as_float((uint32_t)rg[i] << 16);
            g[8 * q + 2 * i + 1] = __uint_as_float((uint32_t)rg[i] & 0xFFFF0000u);
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const v4i rv = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const float*>(h) + ev + 4 * q));
          const v4i rg = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const float*>(h) + eg + 4 * q));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[4 * q + i] = __int_as_float(rv[i]);
            g[4 * q + i] = __int_as_float(rg[i]);
          }
        }
      }
    } else {
      v[0] = BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(h)[ev]) : reinterpret_cast<const float*>(h)[ev];
      g[0] = BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(h)[eg]) : reinterpret_cast<const float*>(h)[eg];
    }
    int code[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const float a = __fmul_rn(v[i], activate(SQ_ACT_GELU, g[i]));
      const bool ng = dual && (a < 0.0f);                 // X_- = min(X, 0) takes the s_- branch of Q_dual
      code[i] = clip_code(round_quotient(a, ng ? sn : sp, ng ? in : ip));
    }
    if (VEC) {
      v4i out;
#pragma unroll
      for (int q = 0; q < 4; ++q) out[q] = (int)pack4(code[4 * q], code[4 * q + 1], code[4 * q + 2], code[4 * q + 3]);
      *reinterpret_cast<v4i*>(xq + m * (size_t)K + col) = out;
    } else {
      xq[m * (size_t)K + col] = (int8_t)code[0];
    }
  }
}

// bf16 input, aligned: GELU(gate) by table.  A bf16 gate has 2^16 bit patterns, and all but a sliver of a layer's gates have
// magnitudes in [2^-14, 8): the results for the kGegluExps * 128 * 2 patterns of that window (17 KiB of fp32, computed by each
// workgroup with activate(), i.e. the very bits the arithmetic path produces) sit in LDS, and a gate costs one ds_read_b32
// instead of the ~35-instruction sequence.  An item with a gate outside the window (tiny, huge, non-finite: seen on the
// packed extremes of its magnitudes) goes through the sequence, in a block of its own so that the common path stays free of
// it.  HBM-bound, 5 bytes per output: 4096 x 5120 21.4 us (4.9 TB/s).  Each by itself: window test on packed extremes instead of
// per element 24.7 -> 23.5 us, items of eight instead of sixteen (which left 2.5 rounds to a thread) 23.5 -> 21.4.  With the layer's
// product behind it, calls in a row, what counts is the sum: 4096 x 5120 x 1280 78.0 -> 74.0 us, 798 x 11264 x 2816 74.0 -> 71.4,
// 1136 x 8704 x 2176 64.6 -> 62.2, 995 x 11776 x 2944 83.6 -> 82.3.  Requesting the first item's loads under the fill of the table and
// every next one's ahead takes the quantizer to 20.9 us, but those sums to 77.5, 77.1, 66.2 and 86.5 on most cards (72.5, 70.7,
// 61.8 and 81.8 on the quickest); ahead in the loop alone, or with one workgroup per CU, is between the two: loads in the loop's
// order are never behind the sixteen-output form.  Persistent workgroups (two per CU) so that
// filling the table is a small part of their work.
constexpr int kGegluExpLo = 113, kGegluExps = 17;        // biased exponents 113 ... 129: 2^-14 <= |gate| < 2^3
constexpr int kGegluThreads = 1024;
__global__ __launch_bounds__(kGegluThreads, 8) void quantize_act_geglu_tab_kernel(const uint16_t* __restrict__ h,
                                                                                  int8_t* __restrict__ xq, int M, int K,
                                                                                  const ActTable tb) {
#pragma clang fp contract(off)
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  constexpr uint32_t LOW = kGegluExpLo << 7, N = kGegluExps * 128;  // window of gate magnitudes, per sign
  __shared__ float gelu_tab[2 * N];
  // items of eight outputs: one 16-byte load of values and one of gates
  const uint32_t per_row = (uint32_t)K >> 3, nitem = (uint32_t)M * per_row;        // M * K < 2^31 (checked by the host)
  const uint32_t stride = gridDim.x * (uint32_t)kGegluThreads, dr = stride / per_row, dc = stride - dr * per_row;
  uint32_t c = blockIdx.x * (uint32_t)kGegluThreads + threadIdx.x, m = c / per_row, cc = c - m * per_row;
  for (int i = threadIdx.x; i < (int)(2 * N); i += kGegluThreads) {
    const uint32_t sign = (uint32_t)i / N, bits = (sign << 15) | (LOW + (uint32_t)i - sign * N);
    gelu_tab[i] = activate(SQ_ACT_GELU, __uint_as_float(bits << 16));
  }
  __syncthreads();
  while (c < nitem) {
    const int col = (int)(8 * cc);
    const uint16_t* p = h + (size_t)m * 2 * (size_t)K + col;
    const v4i cv = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
    const v4i cg = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p + K));
    int8_t* to = xq + (size_t)m * (size_t)K + col;
    c += stride;
    m += dr;
    cc += dc;
    if (cc >= per_row) { cc -= per_row; ++m; }
    float sp = tb.s_pos[0], sn = tb.s_neg[0], ip = tb.inv_pos[0], in = tb.inv_neg[0];
    bool dual = tb.dual[0] != 0;
    for (int s = 1; s < tb.S; ++s) {
      if (col >= tb.kseg_off[s]) {
        sp = tb.s_pos[s]; sn = tb.s_neg[s]; ip = tb.inv_pos[s]; in = tb.inv_neg[s]; dual = tb.dual[s] != 0;
      }
    }
    u16x2 top = {0, 0}, bot = {0xFFFF, 0xFFFF};                     // largest and smallest gate magnitudes of the item
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const u16x2 mag = __builtin_bit_cast(u16x2, (uint32_t)cg[d] & 0x7FFF7FFFu);
      top = __builtin_elementwise_max(top, mag);
      bot = __builtin_elementwise_min(bot, mag);
    }
    float g[8];
    if (top[0] < LOW + N && top[1] < LOW + N && bot[0] >= LOW && bot[1] >= LOW) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t u = (uint32_t)cg[i >> 1], mag = (i & 1) ? (u >> 16) & 0x7FFFu : u & 0x7FFFu;
        const uint32_t neg = ((i & 1) ? u >> 31 : (u >> 15) & 1u) * N;
        g[i] = gelu_tab[mag + neg - LOW];
      }
    } else {                                                        // rare: the whole item by the sequence
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t u = (uint32_t)cg[i >> 1];
        g[i] = activate(SQ_ACT_GELU, __uint_as_float((i & 1) ? u & 0xFFFF0000u : u << 16));
      }
    }
    int out[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      int code[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t u = (uint32_t)cv[2 * q + (i >> 1)];
        const float a = __fmul_rn(__uint_as_float((i & 1) ? u & 0xFFFF0000u : u << 16), g[4 * q + i]);
        const bool neg = dual && (a < 0.0f);
        code[i] = clip_code(round_quotient(a, neg ? sn : sp, neg ? in : ip));
      }
      out[q] = (int)pack4(code[0], code[1], code[2], code[3]);
    }
    *reinterpret_cast<v2i*>(to) = (v2i){out[0], out[1]};
  }
}

hipError_t launch_quantize_act_geglu(const void* h, bool h_is_bf16, int8_t* xq, int M, int K, const ActTable& tb, int cus,
                                     hipStream_t st) {
  bool vec = K % 16 == 0 && (reinterpret_cast<uintptr_t>(h) | reinterpret_cast<uintptr_t>(xq)) % 16 == 0;
  for (int s = 0; s <= tb.S; ++s) vec = vec && tb.kseg_off[s] % 16 == 0;
  const size_t nitem = (size_t)M * (size_t)(vec ? K / 16 : K);
  if (nitem == 0) return hipSuccess;
  // 32768 outputs per compute unit pay for the tables.  Table / direct in us: 820 x 5120 (16400 per compute unit) 8.1 / 7.7, 1024 x
  // 5120 8.7 / 8.4, 1229 x 5120 9.2 / 9.9, 1638 x 5120 (32760, the most that goes direct) 11.1 / 12.3, 2048 x 5120 12.7 / 15.4.
  if (vec && h_is_bf16 && nitem >= (size_t)cus * 2 * kGegluThreads) {
    hipLaunchKernelGGL(quantize_act_geglu_tab_kernel, dim3((unsigned)cus * 2), dim3(kGegluThreads), 0, st,
                       reinterpret_cast<const uint16_t*>(h), xq, M, K, tb);
    return hipGetLastError();
  }
  size_t blocks = (nitem + 255) / 256;
  const size_t cap = (size_t)cus * 64;
  if (blocks > cap) blocks = cap;
#define SQ_G(B, V) hipLaunchKernelGGL((quantize_act_geglu_kernel<B, V>), dim3((unsigned)blocks), dim3(256), 0, st, h, xq, M, K, tb)
  if (h_is_bf16) { if (vec) SQ_G(true, true); else SQ_G(true, false); }
  else           { if (vec) SQ_G(false, true); else SQ_G(false, false); }
#undef SQ_G
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// 4-bit weights (App. B: per-channel weights in the 4-bit settings): the Sec. 3 quantizer with q_max = 7 per output
// channel and K-segment, codes packed two per byte in the order the weight stream consumes them: rows in groups
// of 16 (the last group padded with zero rows), K in steps of 128 codes (T = K / 128), one contiguous KiB per
// (group, step):  packed[((g T + t) 16 + r) 64 + j] = code(16 g + r, 128 t + j) | code(16 g + r, 128 t + 64 + j) << 4
// (4-bit two's complement).  Shifting a fetched dword left by four and masking gives the 16-fold int8 codes of one
// 64-wide MFMA k-step, masking alone those of the next.  One wavefront per (output channel, K-segment); K and the
// segment boundaries are multiples of 128.  Rows beyond N in the last group are zeroed by their own wavefronts.
// ------------------------------------------------------------------------------------------------
template <bool BF16>
__global__ __launch_bounds__(256) void quantize_weight_w4_kernel(const void* __restrict__ w, uint8_t* __restrict__ wq4,
                                                                 float* __restrict__ wscale, int N, int K,
                                                                 const KsegTable tb) {
  const int lane = threadIdx.x & 63;
  const int npad = (N + 15) & ~15;
  const long item = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= (long)npad * tb.S) return;         // whole wave leaves together
  const int n = (int)(item / tb.S), ks = (int)(item % tb.S);
  int k0 = 0, k1 = 0;
  for (int s = 0; s < tb.S; ++s)
    if (s == ks) { k0 = tb.off[s]; k1 = tb.off[s + 1]; }
  const int T = K >> 7;
  uint8_t* out = wq4 + ((size_t)(n >> 4) * T * 16 + (n & 15)) * 64 + lane;      // + t * 1024 per step
  if (n >= N) {                                  // padding row of the last group
    for (int b = k0; b < k1; b += 128) out[(size_t)(b >> 7) * 1024] = 0;
    return;
  }
  const size_t row = (size_t)n * K;
  float a = 0.0f;
  for (int k = k0 + lane; k < k1; k += 64) a = __builtin_fmaxf(a, __builtin_fabsf(load_w<BF16>(w, row + k)));
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) a = __builtin_fmaxf(a, __shfl_xor(a, off, 64));
  const float sw = (a == 0.0f) ? 1.0f : a / 7.0f;
  if (lane == 0) wscale[(size_t)ks * N + n] = sw;
  for (int b = k0; b < k1; b += 128) {
    const float lo = __builtin_fminf(__builtin_fmaxf(__builtin_rintf(load_w<BF16>(w, row + b + lane) / sw), -7.0f), 7.0f);
    const float hi = __builtin_fminf(__builtin_fmaxf(__builtin_rintf(load_w<BF16>(w, row + b + 64 + lane) / sw), -7.0f), 7.0f);
    out[(size_t)(b >> 7) * 1024] = (uint8_t)(((int)lo & 0xF) | (((int)hi & 0xF) << 4));
  }
}

hipError_t launch_quantize_weight_w4(const void* w, bool w_is_bf16, uint8_t* wq4, float* wscale, int N, int K,
                                     const KsegTable& tb, hipStream_t st) {
  if (launch_weight_rows<4>(w, w_is_bf16, wq4, wscale, N, K, tb, st)) return hipGetLastError();
  const long items = (long)((N + 15) & ~15) * tb.S;
  const unsigned blocks = (unsigned)((items + 3) / 4);
  if (w_is_bf16) hipLaunchKernelGGL((quantize_weight_w4_kernel<true>), dim3(blocks), dim3(256), 0, st, w, wq4, wscale, N, K, tb);
  else           hipLaunchKernelGGL((quantize_weight_w4_kernel<false>), dim3(blocks), dim3(256), 0, st, w, wq4, wscale, N, K, tb);
  return hipGetLastError();
}

// Packed 4-bit codes back to one int8 code per byte, [N][K] row-major: what the large-M tile kernel consumes (there the
// GEMM is MFMA-bound and 4-bit weights save memory, not time; a caller unpacks a layer into a reusable buffer right
// before its GEMM).  One thread per 16 packed bytes: the low nibbles are 16 consecutive codes of one row, the high nibbles
// the 16 codes 64 columns further on.  Sign extension of a nibble u per byte: u | (u & 8) * 0x1E.
__global__ __launch_bounds__(256) void unpack_w4_kernel(const uint8_t* __restrict__ wq4, int8_t* __restrict__ wq, int N, int K) {
  const int T = K >> 7;
  const long nitem = (long)((N + 15) >> 4) * T * 16 * 4;           // (group, step, row, 16-byte chunk)
  for (long c = blockIdx.x * 256L + threadIdx.x; c < nitem; c += (long)gridDim.x * 256) {
    const int q = (int)(c & 3), r = (int)((c >> 2) & 15);
    const long gt = c >> 6;
    const int t = (int)(gt % T);
    const long n = (gt / T) * 16 + r;
    if (n >= N) continue;                                          // rows of the last group beyond N hold padding
    const v4i p = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(wq4) + c);
    v4i lo, hi;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t ul = (uint32_t)p[d] & 0x0F0F0F0Fu, uh = ((uint32_t)p[d] >> 4) & 0x0F0F0F0Fu;
      lo[d] = (int)(ul | ((ul & 0x08080808u) * 0x1Eu));
      hi[d] = (int)(uh | ((uh & 0x08080808u) * 0x1Eu));
    }
    int8_t* dst = wq + n * K + 128 * t + 16 * q;
    *reinterpret_cast<v4i*>(dst) = lo;
    *reinterpret_cast<v4i*>(dst + 64) = hi;
  }
}

hipError_t launch_unpack_w4(const uint8_t* wq4, int8_t* wq, int N, int K, int cus, hipStream_t st) {
  const long nitem = (long)((N + 15) >> 4) * (K >> 7) * 64;
  if (nitem == 0) return hipSuccess;
  long blocks = (nitem + 255) / 256;
  if (blocks > (long)cus * 32) blocks = (long)cus * 32;
  hipLaunchKernelGGL(unpack_w4_kernel, dim3((unsigned)blocks), dim3(256), 0, st, wq4, wq, N, K);
  return hipGetLastError();
}

}  // namespace sq
