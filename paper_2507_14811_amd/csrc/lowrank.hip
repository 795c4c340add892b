// Low-rank side branch of the 4-bit settings (main results, W4A8 rows; App. B: SVDQuant is the optimizer of the 4-bit
// settings, rank fixed at 64).  The weight is W = Lu Ld + R; the residual R is quantized and runs through the SegLinear
// kernels, the rank-r part stays in 16 bit on the unquantized activations:
//   y[m][n] = y_q[m][n] + sum_j T[m][j] Lu[n][j],    T[m][j] = sum_k X[m][k] Ld[j][k]        (Ld [r][K], Lu [N][r]).
// Three kernels:
//   * down projection T = X Ld^T on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation): one pass over
//     X, HBM-bound (2 bytes per activation).  bf16 activations with K % 64 == 0 are staged through LDS by direct loads of whole
//     128-byte row pieces, few rows per workgroup, with all of K as a rule; everything else is read straight into fragments.
//     Where there are too few rows to fill the chip K is cut into slices, each of which writes its own fp32 partial T (no
//     atomics: the sum order is fixed).
//   * the slices, if any, summed in ascending order (fp32).
//   * up projection and add: T times Lu^T on the bf16 matrix cores with every fp32 T value split exactly into three bf16
//     terms (T is not rounded to 16 bit), added to y_q before the single rounding to the output type: one read of y_q,
//     one write of y, both in whole row pieces.
#include "sq_kernels.hpp"

namespace sq {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kLrRowsPerWg = 256;     // down projection: 4 waves x 64 token rows
constexpr int kLrMaxSplit = 32;
int lowrank_splits(int M, int K, int cus) {
  const int row_blocks = (M + kLrRowsPerWg - 1) / kLrRowsPerWg;
  int s = (2 * cus + row_blocks - 1) / row_blocks;          // about two workgroups per compute unit
  const int max_by_k = K / 256 > 0 ? K / 256 : 1;          // slices of at least 256 features
  s = s < max_by_k ? s : max_by_k;
  s = s < kLrMaxSplit ? s : kLrMaxSplit;
  return s < 1 ? 1 : s;
}

// A wave owns 64 token rows (two 32-row blocks that share every Ld fragment it fetches) and walks its K slice in
// groups of four 16-feature steps (a lane then reads 128 contiguous bytes of each of its rows per group).  The loads of
// group g + 1 are issued before the matrix instructions of group g, so a wave keeps two groups of loads in flight.
template <bool BF16X, int JB>
__global__ __launch_bounds__(256) void lowrank_down_kernel(const void* __restrict__ x, const uint16_t* __restrict__ ld,
                                                           float* __restrict__ tpart, int M, int K, int slice) {
  constexpr int IM = 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kg = lane >> 5;
  const int k_begin = blockIdx.y * slice;
  const int k_end = (k_begin + slice) < K ? (k_begin + slice) : K;
  int mrow[IM];
  size_t xrow[IM];
#pragma unroll
  for (int i = 0; i < IM; ++i) {
    mrow[i] = blockIdx.x * kLrRowsPerWg + wave * (32 * IM) + i * 32 + (lane & 31);
    xrow[i] = (size_t)(mrow[i] < M ? mrow[i] : M - 1) * K;      // rows beyond M re-read the last row, masked at the store
  }
  v16f acc[IM][JB];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) acc[i][jb] = (v16f)(0.0f);
  auto load_x = [&](const int i, const int k0) __attribute__((always_inline)) {
    if (BF16X) {
      const v4i raw = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(reinterpret_cast<const uint16_t*>(x) + xrow[i] + k0));
      return __builtin_bit_cast(v8bf, raw);
    }
    // fp32 activations enter the 16-bit branch rounded to bf16
    const v4f lo = *reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(x) + xrow[i] + k0);
    const v4f hi = *reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(x) + xrow[i] + k0 + 4);
    v4i p;
    p[0] = (int)f32x2_to_bf16x2(lo[0], lo[1]); p[1] = (int)f32x2_to_bf16x2(lo[2], lo[3]);
    p[2] = (int)f32x2_to_bf16x2(hi[0], hi[1]); p[3] = (int)f32x2_to_bf16x2(hi[2], hi[3]);
    return __builtin_bit_cast(v8bf, p);
  };
  auto load_l = [&](const int jb, const int k0) __attribute__((always_inline)) {
    return *reinterpret_cast<const v8bf*>(ld + (size_t)(jb * 32 + (lane & 31)) * K + k0);
  };
  v8bf xa[2][4][IM], lb[2][4][JB];
  auto load_group = [&](const int buf, const int k) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int i = 0; i < IM; ++i) xa[buf][t][i] = load_x(i, k + 16 * t);
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) lb[buf][t][jb] = load_l(jb, k + 16 * t);
    }
  };
  auto mul_group = [&](const int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
          acc[i][jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lb[buf][t][jb], xa[buf][t][i], acc[i][jb], 0, 0, 0);
  };
  int k = k_begin + 8 * kg;
  const int ngroups = (k_end - k_begin) / 64;                    // whole groups of four steps
  if (ngroups > 0) {
    load_group(0, k);
    int g = 0;
    // the scheduling barriers keep the order written here: all loads of the next group go out before the matrix
    // instructions of the current one (left alone, the compiler sinks each load to just in front of its use)
    for (; g + 2 < ngroups; g += 2) {                            // two groups per trip: the buffer index stays static
      load_group(1, k + 64);
      __builtin_amdgcn_sched_barrier(0);
      mul_group(0);
      __builtin_amdgcn_sched_barrier(0);
      load_group(0, k + 128);
      __builtin_amdgcn_sched_barrier(0);
      mul_group(1);
      __builtin_amdgcn_sched_barrier(0);
      k += 128;
    }
    if (g + 1 < ngroups) {
      load_group(1, k + 64);
      __builtin_amdgcn_sched_barrier(0);
      mul_group(0);
      mul_group(1);
      k += 128;
    } else {
      mul_group(0);
      k += 64;
    }
  }
  for (; k < k_end; k += 16) {                                   // fewer than four steps left
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
      const v8bf l = load_l(jb, k);
#pragma unroll
      for (int i = 0; i < IM; ++i) acc[i][jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l, load_x(i, k), acc[i][jb], 0, 0, 0);
    }
  }
  // element v of block (i, jb) in lane l: row mrow[i], column j = 32 jb + 8 (v >> 2) + 4 (l >> 5) + (v & 3)
#pragma unroll
  for (int i = 0; i < IM; ++i) {
    if (mrow[i] >= M) continue;
    float* out = tpart + ((size_t)blockIdx.y * M + mrow[i]) * (JB * 32);
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4f o = {acc[i][jb][4 * g], acc[i][jb][4 * g + 1], acc[i][jb][4 * g + 2], acc[i][jb][4 * g + 3]};
        *reinterpret_cast<v4f*>(out + jb * 32 + 8 * g + 4 * kg) = o;
      }
  }
}

// The same product for bf16 activations with K % 64 == 0, staged through LDS: a workgroup owns RB = 1, 2 or 4 blocks of 32
// token rows, a stage is 64 features (128 bytes) of those rows and of the rank rows of Ld, fetched with direct global->LDS loads whose
// lanes cover whole 128-byte row pieces (eight rows per instruction) into a ring of NS stages, one barrier per stage.  The four
// waves of a row block take one 16-feature step of every stage each and add their sums through LDS at the end, in a fixed
// order.  The 16-byte chunks of a row are XOR-swizzled with (row >> 1) & 7, which makes the fragment reads (lane -> row lane % 32,
// chunk 2 wave + lane / 32) free of bank conflicts.
// What bounds it is latency: a compute unit moves its ring's bytes once per trip to memory (2.5 us with the chip loaded), so
// the ring takes the whole LDS.  Few rows per workgroup fill the chip with whole rows of X: K is not cut over workgroups, and
// no partial T goes through memory, where a slice of K would be short.
__device__ __forceinline__ void lr_glds16(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

template <int I, int LT>
__device__ __forceinline__ void lr_wait_stages(int left) {      // until at most `left` (<= I) later stages are outstanding
  if constexpr (I == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    if (left >= I) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(I * LT) : "memory");
    else lr_wait_stages<I - 1, LT>(left);
  }
}

template <int JB, int RB, int NS>
__global__ __launch_bounds__(RB * 256) void lowrank_down_lds_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ ld,
                                                               float* __restrict__ tpart, int M, int K, int nsplit) {
  constexpr int R = JB * 32;
  constexpr int ROWS = RB * 32, STAGE = (ROWS + R) * 128;
  // direct loads per wave and stage (8 rows each): one of X and GL of Ld, these by the first LW waves only
  constexpr int GL = R / 8 / (4 * RB) > 0 ? R / 8 / (4 * RB) : 1, LW = R / 8 / GL;
  static_assert(LW <= 4 * RB, "pieces of Ld");
  __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this workgroup's run of 64-feature stages: the K / 64 stages are dealt evenly over the nsplit slices
  const int nst_all = K >> 6, per = nst_all / nsplit, rem = nst_all - per * nsplit;
  const int b = blockIdx.y;
  const int st_begin = b * per + (b < rem ? b : rem);
  const int nst = per + (b < rem ? 1 : 0);
  const int m0 = blockIdx.x * ROWS;

  // direct loads: lane -> (row lane / 8 of the instruction's eight rows, slot lane % 8 holding chunk slot ^ swizzle(row))
  const int lrow = lane >> 3, lslot = lane & 7;
  auto offset = [&](const int rt, const int row) __attribute__((always_inline)) {
    return ((uint32_t)row * (uint32_t)K) * 2u + (uint32_t)((lslot ^ ((rt >> 1) & 7)) << 4);
  };
  const int rx = wave * 8 + lrow;
  const uint32_t voffX = offset(rx, m0 + rx < M ? m0 + rx : M - 1);        // rows beyond M re-read the last row, masked at the store
  const bool with_ld = LW == 4 * RB || wave < LW;
  uint32_t voffL[GL];
#pragma unroll
  for (int g = 0; g < GL; ++g) voffL[g] = offset((wave * GL + g) * 8 + lrow, (wave * GL + g) * 8 + lrow);
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)smem);
  const uint32_t ldsX = lds0 + (uint32_t)wave * 1024u;
  const uint32_t ldsL = lds0 + (uint32_t)ROWS * 128u + (uint32_t)(wave * GL) * 1024u;
  auto issue_stage = [&](const int s) __attribute__((always_inline)) {       // s: stage index inside this slice
    const size_t kbyte = (size_t)(st_begin + s) * 128;
    // uniform base addresses in scalar registers (the halves go through unsigned 32-bit values: readfirstlane returns a
    // signed int, which would be sign-extended into the upper half)
    auto uniform_ptr = [](const uint16_t* p, size_t byte_off) __attribute__((always_inline)) {
      const uint64_t u = reinterpret_cast<uint64_t>(p) + byte_off;
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)u);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
      return reinterpret_cast<const void*>(((uint64_t)hi << 32) | (uint64_t)lo);
    };
    const void* px = uniform_ptr(x, kbyte);
    const void* pl = uniform_ptr(ld, kbyte);
    const uint32_t so = __builtin_amdgcn_readfirstlane((uint32_t)(s % NS) * (uint32_t)STAGE);
    lr_glds16(px, voffX, __builtin_amdgcn_readfirstlane(ldsX + so));
    if (with_ld)
#pragma unroll
      for (int g = 0; g < GL; ++g) lr_glds16(pl, voffL[g], __builtin_amdgcn_readfirstlane(ldsL + so + (uint32_t)g * 1024u));
  };

  // fragments: row lane % 32 of a 32-row block, chunk 2 kw + lane / 32
  const int kw = wave & 3, rb = wave >> 2;
  const int frow = lane & 31, fhi = lane >> 5;
  const int foff = frow * 128 + (((2 * kw + fhi) ^ ((frow >> 1) & 7)) << 4);
  v16f acc[JB];
#pragma unroll
  for (int jb = 0; jb < JB; ++jb) acc[jb] = (v16f)(0.0f);

#pragma unroll 1
  for (int s = 0; s < NS - 1 && s < nst; ++s) issue_stage(s);
#pragma unroll 1
  for (int s = 0; s < nst; ++s) {
    // stage s has landed in this wave's view (loads return in order)
    if (with_ld) lr_wait_stages<NS - 2, 1 + GL>(nst - 1 - s);
    else lr_wait_stages<NS - 2, 1>(nst - 1 - s);
    __syncthreads();                                          // ... and in every wave's; the buffer of stage s - 1 is free
    if (s + NS - 1 < nst) issue_stage(s + NS - 1);
    const char* frag = smem + (s % NS) * STAGE + foff;
    const v8bf xa = *reinterpret_cast<const v8bf*>(frag + rb * (32 * 128));
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
      const v8bf lb = *reinterpret_cast<const v8bf*>(frag + (ROWS + jb * 32) * 128);
      acc[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lb, xa, acc[jb], 0, 0, 0);
    }
  }
  // element v of block jb in lane l: row m0 + 32 rb + (l & 31), column j = 32 jb + 8 (v >> 2) + 4 (l >> 5) + (v & 3).  Run q = 4 jb +
  // (v >> 2) of four columns is added up by wave q / JB of the row block, in the order of the waves.
  static_assert(4 * RB * 4 * JB * 1024 <= NS * STAGE, "the sums of all waves");
  __syncthreads();                                            // the ring has been read
  char* sums = smem + rb * (16 * JB * 1024) + lane * 16;
#pragma unroll
  for (int q = 0; q < 4 * JB; ++q) {
    const v16f& t = acc[q >> 2];
    const int v = 4 * (q & 3);
    *reinterpret_cast<v4f*>(sums + (kw * 4 * JB + q) * 1024) = (v4f){t[v], t[v + 1], t[v + 2], t[v + 3]};
  }
  __syncthreads();
  const int m = m0 + rb * 32 + frow;
  if (m >= M) return;
  float* out = tpart + ((size_t)blockIdx.y * M + m) * R;
#pragma unroll
  for (int i = 0; i < JB; ++i) {
    const int q = kw * JB + i;
    v4f sum = *reinterpret_cast<const v4f*>(sums + q * 1024);
#pragma unroll
    for (int w = 1; w < 4; ++w) sum += *reinterpret_cast<const v4f*>(sums + (w * 4 * JB + q) * 1024);
    *reinterpret_cast<v4f*>(out + 8 * q + 4 * fhi) = sum;
  }
}

// Row blocks per workgroup and slices of K: the choice that moves the fewest bytes into a compute unit.  The launch of the sum costs
// what moves in 2 - 3 us (144 KB), and a byte of partial T, written and read back by all at once, as much as ten of a ring.  8500 x
// 1536, rank 64: 256 rows and seven slices took 10.6 + 5.3 us for the sum, two row blocks and no slices take 13.1.  Whole call with
// N = 128, 160 sizes of 1 - 16384 rows and K of 512 - 16384, against 256 rows and a workgroup per compute unit always: 4096 x 1536
// 17.9 -> 15.5 us, 256 x 3072 16.0 -> 14.2, 64 x 8192 20.3 -> 16.5, 6000 x 3072 22.2 -> 19.7; 8500 x 4096 27.9 -> 28.4 is the worst.
struct DownPlan { int rb, slices; };
constexpr int kLdsSliceStages = 8, kLdsRing = 144 * 1024;
static DownPlan lowrank_lds_plan(int M, int K, int rank, int cus) {
  DownPlan best{1, 1};
  long long least = -1;
  const int nst = K >> 6;
  for (int rb = 1; rb <= 4; rb *= 2) {
    const int blocks = (M + 32 * rb - 1) / (32 * rb);
    int most = cus / blocks;                                     // slices of at least eight stages, a workgroup per compute unit
    most = most < nst / kLdsSliceStages ? most : nst / kLdsSliceStages;
    most = most < kLrMaxSplit ? most : kLrMaxSplit;
    for (int pass = 0; pass < 2; ++pass) {
      const int s = pass == 0 || most < 1 ? 1 : most;
      const long long rounds = (blocks * s + cus - 1) / cus;
      const long long cost = rounds * ((nst + s - 1) / s) * ((32 * rb + rank) * 128) + (s > 1 ? 144 * 1024 + 40ll * s * M * rank / cus : 0);
      if (least < 0 || cost < least) { least = cost; best = {rb, s}; }
    }
  }
  return best;
}
template <int JB>
static void launch_down_lds(const uint16_t* x, const uint16_t* ld, float* tpart, int M, int K, DownPlan p, hipStream_t st) {
#define SQ_DOWN(RB) hipLaunchKernelGGL((lowrank_down_lds_kernel<JB, RB, (kLdsRing / ((32 * RB + 32 * JB) * 128) < 12 ? kLdsRing / ((32 * RB + 32 * JB) * 128) : 12)>), dim3((M + 32 * RB - 1) / (32 * RB), p.slices), dim3(RB * 256), 0, st, x, ld, tpart, M, K, p.slices)
  if (p.rb == 1) SQ_DOWN(1);
  else if (p.rb == 2) SQ_DOWN(2);
  else SQ_DOWN(4);
#undef SQ_DOWN
}
static bool lowrank_lds_usable(const void* x, bool x_is_bf16, const uint16_t* ld, int M, int K) {
  return x_is_bf16 && K % 64 == 0 && K >= 64 && (size_t)M * K * 2 < 0x7FFFFFFFull && (size_t)64 * K * 2 < 0x7FFFFFFFull &&
         (reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(ld)) % 16 == 0;
}

// T = sum of the K slices' partial results, in ascending slice order (fp32): four values per thread.
__global__ __launch_bounds__(256) void lowrank_sum_kernel(const float* __restrict__ tpart, int nsplit, size_t nvec, float* __restrict__ tsum) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nvec) return;
  v4f s = reinterpret_cast<const v4f*>(tpart)[i];
  for (int sp = 1; sp < nsplit; ++sp) s += reinterpret_cast<const v4f*>(tpart)[(size_t)sp * nvec + i];
  reinterpret_cast<v4f*>(tsum)[i] = s;
}

// KH consecutive features of T, split exactly into three bf16 terms (hi + mid + lo carries the 24-bit mantissa; the last term is
// rounded at 2^-25 of the value), eight features per matrix instruction
template <int KH>
__device__ __forceinline__ void split_t(const float* src, v8bf (&thi)[KH / 8], v8bf (&tmid)[KH / 8], v8bf (&tlo)[KH / 8]) {
#pragma unroll
  for (int c = 0; c < KH / 8; ++c) {
    const v4f a = *reinterpret_cast<const v4f*>(src + 8 * c), b = *reinterpret_cast<const v4f*>(src + 8 * c + 4);
    const float t[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    v4i ph, pm, pl;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t hb = f32x2_to_bf16x2(t[2 * i], t[2 * i + 1]);
      const float r0 = t[2 * i] - __uint_as_float(hb << 16), r1 = t[2 * i + 1] - __uint_as_float(hb & 0xFFFF0000u);
      const uint32_t mbits = f32x2_to_bf16x2(r0, r1);
      const float q0 = r0 - __uint_as_float(mbits << 16), q1 = r1 - __uint_as_float(mbits & 0xFFFF0000u);
      ph[i] = (int)hb;
      pm[i] = (int)mbits;
      pl[i] = (int)f32x2_to_bf16x2(q0, q1);
    }
    thi[c] = __builtin_bit_cast(v8bf, ph);
    tmid[c] = __builtin_bit_cast(v8bf, pm);
    tlo[c] = __builtin_bit_cast(v8bf, pl);
  }
}

// Up projection and addition.  A wave owns 32 token rows: its T fragment stays in registers as three bf16 terms per value, Lu rows
// (bf16) are the other operand, one 32 x 32 block of outputs at a time, three v_mfma_f32_32x32x16_bf16 per 16 features (fp32
// accumulation; 12 matrix instructions per block for rank 64 where the fp32 instruction v_mfma_f32_32x32x2_f32 needs 32 of twice
// the length).  The matrix instruction pairs lane half h of both operands, so half h takes the features [h R/2, (h + 1) R/2) of T
// and Lu.  T is the "A" operand: a half-wave then holds 32 consecutive columns of one row.
// What bounds it is memory: y_q is read and y written once (235 MB at 8500 x 1536 x 4608, 46 us at the rate of a large copy).
//   * A workgroup owns 128 token rows and kLrStrip columns, whose Lu rows it stages in LDS once by direct loads of whole lines; a
//     wave that fetches them itself touches 32 lines per load instruction and fetches them four times as often.
//   * y_q of the next block is requested ahead of the matrix instructions of the current one, except at rank 32 and less than 11 M
//     outputs, where the registers cost a wave per SIMD (6266 x 512 x 1536 48.1 us, without 46.0), and past the caches from 13 M outputs on
//     where rows are whole lines (8500 x 1536 x 4608 153.4 us; 6987 x 1920 x 5418 241 past them, 231 through them).
//   * Where y_q and y together fill half to all of the 256 MB Infinity Cache, y is stored past it as well: ordinary stores displace y_q
//     that has not been read yet.  4-bit layer with the branch (quantizer to y), stores past the cache / ordinary / waves that fetch
//     Lu themselves: 8500 x 1536 x 4608 (235 MB) 148.8 / 154.1 / 160.2 us, 2749 x 2816 x 8448 (139 MB) 126.6 / 127.1 / 133.0, but
//     2236 x 1792 x 5376 (72 MB) 67.3 / 65.1 / 72.6 and 4298 x 4096 x 12288 (317 MB) 306.3 / 301.5 / 303.6.  The lines are in
//     outputs because fp32 y gains in the same range, at a third more bytes: product and branch, y past the cache / only y_q / neither,
//     bf16 27.6 M outputs 104.8 / 107.9 / 115.2 us, 39.2 M (rank 32) 139.5 / 151.2 / 167.0; fp32 27.6 M 112.7 / 115.9 / 120.1, 39.2 M
//     145.9 / 170.0 / 177.6; at 13.2 M and 52.8 M all three within 2 % (fp32 58.1 / 57.7 / 57.8, 314 / 316 / 320).  Without y_q fp32 y
//     gains from 15 M on (33.0 M 47.2 / 53.4), bf16 y 2 - 3 %.
// Measured and not taken: 16-byte accesses (a load covers 64 bytes of 16 rows instead of 128 of two; 170 - 179 us), strips of 256
// columns (152.3).
constexpr int kLrStrip = 128;
constexpr long long kLrAhead = 11000000, kLrReadPast = 13000000, kLrPastFrom = 20000000, kLrPastTo = 44000000;   // outputs
enum LrMode { LR_SHORT, LR_AHEAD, LR_READ_PAST, LR_PAST };           // each with what the ones before it have
template <bool YBF16, int R, LrMode MODE>
__global__ __launch_bounds__(256) void lowrank_up_kernel(const float* __restrict__ tsum, const uint16_t* __restrict__ lu,
                                                         const float* y_in, void* y_out, int M, int N) {
  constexpr int KH = R / 2, RB = R * 2;                            // features of a lane half, bytes of a Lu row
  constexpr int SW = RB == 128 ? 7 : 3;
  __shared__ __attribute__((aligned(1024))) char smem[kLrStrip * RB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, frow = lane & 31;
  const int n0 = blockIdx.x * kLrStrip;
  const int ncols = (N - n0) < kLrStrip ? (N - n0) : kLrStrip;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)smem);
  constexpr int RPI = 1024 / RB, CPR = RB / 16;
  const uint16_t* strip = lu + (size_t)n0 * R;                     // Lu may exceed 4 GiB: 32-bit offsets only inside the strip
#pragma unroll
  for (int g = 0; g < kLrStrip / RPI / 4; ++g) {
    const int rt = (wave * (kLrStrip / RPI / 4) + g) * RPI + lane / CPR;
    const int r = rt < ncols ? rt : ncols - 1;                     // beyond N: re-read the last row, masked at the store
    const int slot = (lane % CPR) ^ ((RB == 128 ? rt >> 1 : rt >> 2) & SW);
    lr_glds16(strip, (uint32_t)(r * RB + (slot << 4)), __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(wave * (kLrStrip / RPI / 4) + g) * 1024u));
  }
  const int mb = blockIdx.y * 128 + wave * 32;
  v8bf thi[KH / 8], tmid[KH / 8], tlo[KH / 8];
  {
    const int m = mb + frow;
    split_t<KH>(tsum + (size_t)(m < M ? m : M - 1) * R + KH * h, thi, tmid, tlo);
  }
  const bool pair_ok = (N % 2 == 0) && (reinterpret_cast<uintptr_t>(y_out) % 4 == 0);     // two bf16 columns per store
  auto store = [](auto* p, const auto v) __attribute__((always_inline)) {
    if (MODE == LR_PAST) __builtin_nontemporal_store(v, p);
    else *p = v;
  };
  // element v of a block in lane l: token row mb + 8 (v >> 2) + 4 (l >> 5) + (v & 3), output column nb + (l & 31): every access covers
  // whole 128-byte (fp32) or 64-byte (bf16) row pieces.  Rows and columns beyond the matrix re-read the last ones.
  struct Yq { float q[16]; };
  auto load_yq = [&](const int nb) __attribute__((always_inline)) {
    Yq t;
    const int n = nb + frow, na = n < N ? n : N - 1;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int mv = mb + 8 * (v >> 2) + 4 * h + (v & 3);
      const float* src = y_in + (size_t)(mv < M ? mv : M - 1) * N + na;
      t.q[v] = y_in == nullptr ? 0.0f : MODE >= LR_READ_PAST ? __builtin_nontemporal_load(src) : *src;
    }
    return t;
  };
  Yq next;
  if (MODE >= LR_AHEAD) next = load_yq(n0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // Lu has landed
  __syncthreads();
  if (mb >= M) return;
#pragma unroll 1
  for (int nb = 0; nb < ncols; nb += 32) {
    Yq cur;
    if (MODE >= LR_AHEAD) {
      cur = next;
      if (nb + 32 < ncols) next = load_yq(n0 + nb + 32);
    } else {
      cur = load_yq(n0 + nb);
    }
    v16f acc = (v16f)(0.0f);
    v8bf lf[KH / 8];
#pragma unroll
    for (int c = 0; c < KH / 8; ++c) {
      const int chunk = (KH / 8) * h + c, r = nb + frow;
      lf[c] = *reinterpret_cast<const v8bf*>(smem + r * RB + ((chunk ^ ((RB == 128 ? r >> 1 : r >> 2) & SW)) << 4));
    }
#pragma unroll
    for (int c = 0; c < KH / 8; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tlo[c], lf[c], acc, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < KH / 8; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tmid[c], lf[c], acc, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < KH / 8; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(thi[c], lf[c], acc, 0, 0, 0);
    const int n = n0 + nb + frow;
    const bool n_ok = n < N;
    if (YBF16 && pair_ok) {
      // bf16: neighbouring lanes exchange one value of every row pair, so that a lane stores two adjacent columns (4 bytes):
      // even lanes the row of element 2 u, odd lanes the row of element 2 u + 1
      const bool odd = (lane & 1) != 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float o0 = cur.q[2 * u] + acc[2 * u], o1 = cur.q[2 * u + 1] + acc[2 * u + 1];
        const float send = odd ? o0 : o1;
        const float recv = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), 0xB1, 0xF, 0xF, false));   // lane ^ 1
        const int v = 2 * u + (odd ? 1 : 0);
        const int mv = mb + 8 * (v >> 2) + 4 * h + (v & 3);
        const uint32_t pk = odd ? f32x2_to_bf16x2(recv, o1) : f32x2_to_bf16x2(o0, recv);
        if (n_ok && mv < M) store(reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(y_out) + (size_t)mv * N + (n & ~1)), pk);
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int mv = mb + 8 * (v >> 2) + 4 * h + (v & 3);
        const float o = cur.q[v] + acc[v];
        if (n_ok && mv < M) {
          if (YBF16) reinterpret_cast<uint16_t*>(y_out)[(size_t)mv * N + n] = f32_to_bf16(o);
          else store(reinterpret_cast<float*>(y_out) + (size_t)mv * N + n, o);
        }
      }
    }
  }
}

size_t lowrank_workspace_bytes(int M, int K, int rank, int cus) {
  const int a = lowrank_splits(M, K, cus), b = lowrank_lds_plan(M, K, rank, cus).slices;    // whichever down projection runs
  return (size_t)((a > b ? a : b) + 1) * M * rank * sizeof(float);               // the slices' partial T, then their sum
}

hipError_t launch_lowrank_add(const void* x, bool x_is_bf16, const uint16_t* ld, const uint16_t* lu, int rank, const float* y_in,
                              void* y_out, bool y_is_bf16, int M, int K, int N, float* workspace, int cus, hipStream_t st) {
  int nsplit;
  if (lowrank_lds_usable(x, x_is_bf16, ld, M, K)) {
    const DownPlan p = lowrank_lds_plan(M, K, rank, cus);
    nsplit = p.slices;
    if (rank == 64) launch_down_lds<2>(reinterpret_cast<const uint16_t*>(x), ld, workspace, M, K, p, st);
    else launch_down_lds<1>(reinterpret_cast<const uint16_t*>(x), ld, workspace, M, K, p, st);
  } else {
    nsplit = lowrank_splits(M, K, cus);
    int slice = (K + nsplit - 1) / nsplit;
    slice = (slice + 63) / 64 * 64;                              // whole groups of four 16-feature steps, except at the end of K
    dim3 gd((M + kLrRowsPerWg - 1) / kLrRowsPerWg, nsplit);
#define SQ_DOWN(B, J) hipLaunchKernelGGL((lowrank_down_kernel<B, J>), gd, dim3(256), 0, st, x, ld, workspace, M, K, slice)
    if (rank == 64) { if (x_is_bf16) SQ_DOWN(true, 2); else SQ_DOWN(false, 2); }
    else            { if (x_is_bf16) SQ_DOWN(true, 1); else SQ_DOWN(false, 1); }
#undef SQ_DOWN
  }
  const float* tsum = workspace;
  if (nsplit > 1) {
    float* dst = workspace + (size_t)nsplit * M * rank;
    const size_t nvec = (size_t)M * rank / 4;
    hipLaunchKernelGGL(lowrank_sum_kernel, dim3((unsigned)((nvec + 255) / 256)), dim3(256), 0, st, workspace, nsplit, nvec, dst);
    tsum = dst;
  }
  const dim3 gu((N + kLrStrip - 1) / kLrStrip, (M + 127) / 128);
  const long long outputs = (long long)M * N;
  const bool lines = N % 32 == 0;                                    // rows begin on whole lines of y_q and 64-byte pieces of bf16 y
#define SQ_UPM(B, R, MODE) hipLaunchKernelGGL((lowrank_up_kernel<B, R, MODE>), gu, dim3(256), 0, st, tsum, lu, y_in, y_out, M, N)
#define SQ_UP(B, R) \
  if (lines && outputs >= kLrPastFrom && outputs < kLrPastTo) SQ_UPM(B, R, LR_PAST); \
  else if (lines && outputs >= kLrReadPast) SQ_UPM(B, R, LR_READ_PAST); \
  else if (R == 64 || outputs >= kLrAhead) SQ_UPM(B, R, LR_AHEAD); \
  else SQ_UPM(B, R, LR_SHORT)
  if (rank == 64) { if (y_is_bf16) { SQ_UP(true, 64); } else { SQ_UP(false, 64); } }
  else            { if (y_is_bf16) { SQ_UP(true, 32); } else { SQ_UP(false, 32); } }
#undef SQ_UP
#undef SQ_UPM
  return hipGetLastError();
}

}  // namespace sq
