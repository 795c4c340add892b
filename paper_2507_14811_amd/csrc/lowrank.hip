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

#include <type_traits>

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
__device__ __forceinline__ void split_t(const v4f (&src)[KH / 4], v8bf (&thi)[KH / 8], v8bf (&tmid)[KH / 8], v8bf (&tlo)[KH / 8]) {
#pragma unroll
  for (int c = 0; c < KH / 8; ++c) {
    const v4f a = src[2 * c], b = src[2 * c + 1];
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
// and Lu.  T is the "A" operand: a lane holds one column of 16 rows.
// What bounds it is memory: y_q is read and y written once (235 MB at 8500 x 1536 x 4608, 46 us at the rate of a large copy).
//   * A lane holds CPL = 4 (or 2) neighbouring columns, one in each of CPL blocks: place 32 j + f of the staged strip holds Lu row
//     CPL f + j, so the order costs nothing.  A load of y_q then covers 512 (256) consecutive bytes of two rows, a store 256 (128)
//     bytes of bf16 y; with a block of 32 neighbouring columns at a time they were 128 and 64, and twice to four times as many.
//   * All loads of a wave (its share of Lu, T, y_q) go out before anything waits; the T values are split meanwhile.  Whether there is a
//     y_q is a template argument: as a branch in the kernel, both sides began with T, and the compiler waited for it in front of the
//     branch (and kept 36 registers more, 16 bytes of them in scratch memory at CPL = 2).  Timed in turn the two orders are alike, other
//     waves fill the gap: 8500 x 1536 x 4608 134.1 -> 133.2 us, 1500 x 1024 x 3072 39.0 -> 38.1, 2749 x 2816 x 8448 117.9 -> 118.2.
//   * Row blocks run from the last to the first: the product has written the last rows of y_q last, and they are still in the Infinity
//     Cache, while the first ones of a large y_q would be displaced before they are read.
//   * Where rows are whole lines, large calls go past the caches; what still fits in the Infinity Cache is quicker through it, and whoever
//     reads y next pays for what does not go there.  bf16 y: y_q and y past them from 10 M outputs on (4-bit layer 5300 x 1024 x 3072 54.2 us,
//     through them 55.2; with a quantizer reading y 67.2 / 67.9; 1100 x 3072 x 9216 72.3 / 72.3, 82.6 / 81.9).  fp32 y: y_q from 13 M on
//     and y from 20 to 44 M (y_q written, this call, y read: 3787 x 2048 x 4032 65.9 us, y past them 69.2; 10 - 20 M 1.02 - 1.06 times as
//     fast in the mean; beyond 44 M alike).  Below, y_q past them took 2 - 5 % longer where it had stayed there, and 0 - 1 % in a layer.  Without
//     a y_q nothing goes past them (20 - 44 M, with a reader, fp32 1.00 - 1.08 and bf16 1.00 - 1.05 times as fast).
// 4-bit layer with the branch (quantizer to y), 32 columns at a time / here with rows upwards / as it is: 8500 x 1536 x 4608 145 / 140 /
// 134.5 us, 2749 x 2816 x 8448 122 / 123 / 116.5, 8191 x 896 x 2688 81 / 81.5 / 77, 7000 x 3072 x 9216 313 / 290 / 290, 6987 x 1920 x
// 5418 225 / 211 / 209 (rows of odd length, through the caches: past them 3 - 7 % slower).
// Not taken: three waves per SIMD at CPL = 4 (the registers spill: 163 us), CPL = 2 throughout (290 -> 302 at 7000 x 3072 x 9216).
constexpr long long kLrPastFromBf16 = 10000000, kLrReadPast = 13000000, kLrPastFrom = 20000000, kLrPastTo = 44000000;   // outputs
enum LrMode { LR_PLAIN, LR_READ_PAST, LR_PAST };                     // each with what the ones before it have
template <bool YBF16, int R, int CPL, LrMode MODE, bool YQ>
__global__ __launch_bounds__(256, CPL == 4 ? 2 : 3) void lowrank_up_kernel(const float* __restrict__ tsum, const uint16_t* __restrict__ lu,
                                                                           const float* y_in, void* y_out, int M, int N) {
  constexpr int STRIP = 32 * CPL;                                  // columns of a workgroup, CPL per lane
  constexpr int KH = R / 2, RB = R * 2;                            // features of a lane half, bytes of a Lu row
  constexpr int SW = RB == 128 ? 7 : 3;
  __shared__ __attribute__((aligned(1024))) char smem[STRIP * RB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, frow = lane & 31;
  const int n0 = blockIdx.x * STRIP;
  const int ncols = (N - n0) < STRIP ? (N - n0) : STRIP;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) char*)smem);
  constexpr int RPI = 1024 / RB, CPR = RB / 16;
  const uint16_t* strip = lu + (size_t)n0 * R;                     // Lu may exceed 4 GiB: 32-bit offsets only inside the strip
#pragma unroll
  for (int g = 0; g < STRIP / RPI / 4; ++g) {
    const int rt = (wave * (STRIP / RPI / 4) + g) * RPI + lane / CPR;   // place 32 j + f holds Lu row CPL f + j
    const int col = CPL * (rt & 31) + (rt >> 5);
    const int r = col < ncols ? col : ncols - 1;                   // beyond N: re-read the last row, masked at the store
    const int slot = (lane % CPR) ^ ((RB == 128 ? rt >> 1 : rt >> 2) & SW);
    lr_glds16(strip, (uint32_t)(r * RB + (slot << 4)), __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(wave * (STRIP / RPI / 4) + g) * 1024u));
  }
  const int mb = (int)(gridDim.y - 1 - blockIdx.y) * 128 + wave * 32;
  // Element v of block j in lane l: token row mb + 8 (v >> 2) + 4 (l >> 5) + (v & 3), output column n0 + CPL (l & 31) + j.  FULL: the
  // wave's rows and the strip lie inside the matrix (addresses are then a scalar per row and one offset per lane); else rows beyond
  // it re-read the last one.
  const int nl = n0 + CPL * frow;
  auto strip_of = [&](auto full_tag) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_tag)::value;
    typedef float vf __attribute__((ext_vector_type(CPL)));
    typedef float vfu __attribute__((ext_vector_type(CPL), aligned(4)));   // rows of any N: 4-byte (bf16: 2-byte) alignment
    typedef int viu __attribute__((ext_vector_type(CPL / 2), aligned(2)));
    const uint32_t here = (uint32_t)(4 * h) * (uint32_t)N + (uint32_t)(CPL * frow);   // FULL: 32 N < 2^31
    auto first_of = [&](const int v) __attribute__((always_inline)) { return (size_t)(mb + 8 * (v >> 2) + (v & 3)) * N + n0; };
    v4f t[KH / 4];
    {
      const int m = mb + frow;
      const v4f* src = reinterpret_cast<const v4f*>(tsum + (size_t)(FULL || m < M ? m : M - 1) * R + KH * h);
#pragma unroll
      for (int c = 0; c < KH / 4; ++c) t[c] = src[c];
    }
    asm volatile("" ::: "memory");                                 // T is requested ahead of y_q
    vf q[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      q[v] = (vf)(0.0f);
      if (YQ && FULL) {
        const vfu* s4 = reinterpret_cast<const vfu*>(reinterpret_cast<const char*>(y_in + first_of(v)) + here * 4u);
        q[v] = MODE >= LR_READ_PAST ? __builtin_nontemporal_load(s4) : *s4;
      } else if (YQ) {
        const int mv = mb + 8 * (v >> 2) + 4 * h + (v & 3);
        const float* src = y_in + (size_t)(mv < M ? mv : M - 1) * N;
#pragma unroll
        for (int j = 0; j < CPL; ++j) q[v][j] = src[nl + j < N ? nl + j : N - 1];
      }
    }
    __builtin_amdgcn_sched_barrier(0);                             // all loads are out
    v8bf thi[KH / 8], tmid[KH / 8], tlo[KH / 8];
    split_t<KH>(t, thi, tmid, tlo);
    // Lu has landed: the sixteen loads of y_q are younger
    if (FULL && YQ) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (!FULL && mb >= M) return;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      v16f acc = (v16f)(0.0f);
      v8bf lf[KH / 8];
#pragma unroll
      for (int c = 0; c < KH / 8; ++c) {
        const int chunk = (KH / 8) * h + c, r = 32 * j + frow;
        lf[c] = *reinterpret_cast<const v8bf*>(smem + r * RB + ((chunk ^ ((RB == 128 ? r >> 1 : r >> 2) & SW)) << 4));
      }
#pragma unroll
      for (int c = 0; c < KH / 8; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tlo[c], lf[c], acc, 0, 0, 0);
#pragma unroll
      for (int c = 0; c < KH / 8; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tmid[c], lf[c], acc, 0, 0, 0);
#pragma unroll
      for (int c = 0; c < KH / 8; ++c) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(thi[c], lf[c], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 16; ++v) q[v][j] += acc[v];
      __builtin_amdgcn_sched_barrier(0);                           // one block's sums at a time
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int mv = mb + 8 * (v >> 2) + 4 * h + (v & 3);
      viu p;
#pragma unroll
      for (int j = 0; j < CPL; j += 2) p[j / 2] = (int)f32x2_to_bf16x2(q[v][j], q[v][j + 1]);
      if constexpr (FULL && YBF16) {
        viu* y = reinterpret_cast<viu*>(reinterpret_cast<char*>(reinterpret_cast<uint16_t*>(y_out) + first_of(v)) + here * 2u);
        if (MODE == LR_PAST) __builtin_nontemporal_store(p, y);
        else *y = p;
      } else if constexpr (FULL) {
        vfu* y = reinterpret_cast<vfu*>(reinterpret_cast<char*>(reinterpret_cast<float*>(y_out) + first_of(v)) + here * 4u);
        const vfu t = q[v];
        if (MODE == LR_PAST) __builtin_nontemporal_store(t, y);
        else *y = t;
      } else if (mv < M) {
#pragma unroll
        for (int j = 0; j < CPL; ++j)
          if (nl + j < N) {
            if (YBF16) reinterpret_cast<uint16_t*>(y_out)[(size_t)mv * N + nl + j] = (uint16_t)((uint32_t)p[j >> 1] >> (16 * (j & 1)));
            else reinterpret_cast<float*>(y_out)[(size_t)mv * N + nl + j] = q[v][j];
          }
      }
    }
  };
  if (ncols == STRIP && mb + 32 <= M) strip_of(std::true_type{});
  else strip_of(std::false_type{});
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
  const bool lines = N % 32 == 0;                                    // rows begin on whole lines of y_q and 64-byte pieces of bf16 y
  // Four columns per lane where their 128 x 128 blocks fill the compute units (two workgroups each); below, half as wide strips spread
  // over more of them: 1500 x 1024 x 3072 39.2 -> 37.5 us, 700 x 1024 x 3072 33.0 -> 31.3, 400 x 3072 x 9216 53.5 -> 51.9.
  const int rows = (M + 127) / 128;
  const bool wide = (long long)rows * ((N + 127) / 128) >= 2ll * cus;
  // Narrow strips have less than 2 cus x 128 x 128 = 8.4 M outputs, and without a y_q y goes through the caches: past them is for wide ones.
  const long long outputs = (long long)M * N;
  const bool y_past = lines && (y_is_bf16 ? outputs >= kLrPastFromBf16 : outputs >= kLrPastFrom && outputs < kLrPastTo);
  const bool read_past = lines && outputs >= kLrReadPast;            // fp32 y; with bf16 y kLrPastFromBf16 is for both
#define SQ_UPM(B, R, C, MODE, YQ) hipLaunchKernelGGL((lowrank_up_kernel<B, R, C, MODE, YQ>), dim3((N + 32 * C - 1) / (32 * C), rows), dim3(256), 0, st, tsum, lu, y_in, y_out, M, N)
#define SQ_UP(B, R) \
  if (y_in == nullptr) { \
    if (wide) SQ_UPM(B, R, 4, LR_PLAIN, false); \
    else SQ_UPM(B, R, 2, LR_PLAIN, false); \
  } else if (!wide) { \
    SQ_UPM(B, R, 2, LR_PLAIN, true); \
  } else if (y_past) { \
    SQ_UPM(B, R, 4, LR_PAST, true); \
  } else if (read_past) { \
    SQ_UPM(B, R, 4, (B ? LR_PLAIN : LR_READ_PAST), true); \
  } else { \
    SQ_UPM(B, R, 4, LR_PLAIN, true); \
  }
  if (rank == 64) { if (y_is_bf16) { SQ_UP(true, 64) } else { SQ_UP(false, 64) } }
  else            { if (y_is_bf16) { SQ_UP(true, 32) } else { SQ_UP(false, 32) } }
#undef SQ_UP
#undef SQ_UPM
  return hipGetLastError();
}

}  // namespace sq
