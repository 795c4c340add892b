// SegLinear + DualScale GEMM for layers with few output tiles (up to about a thousand token rows times a long reduction,
// e.g. the feed-forward down projections of a text stream): small tiles whose waves split K among themselves.
//
// The kernel of seglinear_mfma_kernel.hpp has one wave per SIMD.  On the small tiles that such a layer needs to spread over
// the compute units its waves re-read each other's operand rows from LDS, and a k-step has only 4 - 6 MFMAs under which to
// hide the reads of the next one: 333 x 6144 x 1536 (both polarities) runs on 72 tiles of 64 x 128 at 0.65 us per 128-byte stage,
// of which the MFMAs are 0.21.  Here a workgroup of eight waves (two per SIMD, one wave's LDS reads and separation run under
// the other's MFMAs) owns a tile; four waves share a half of it and take one 32-byte k-step each of every stage.  A stage's
// X^ bytes are then read from LDS once and its W^ bytes twice (64 x 128: the other way round), whatever the tile, and tiles
// can be small.  The price is an exchange of the int32 partial sums through LDS per K-segment (1.5 us for 64 x 64): exact
// integers, so the result does not depend on the split.  Measured: 333 x 6144 x 1536 34.2 -> 16.2 us, 512 x 12288 x 3072
// 62.4 -> 42 us, 106 x 14848 x 3712 75.5 -> 30 us, 70 x 1920 x 5760 (one path) 10.6 -> 7.8 us.
//
// What bounds it: the direct loads (24 KB per stage of a 64 x 128 tile alone take 0.25 us, 100 GB/s and compute unit), next
// to MFMAs of 0.24 us and LDS reads of 0.1 us; all of them together 0.35 - 0.48 us.
//
// Operands arrive by direct global->LDS loads into a ring of NS stages (144 KB), with the swizzle and fragment layout of the
// tile kernel (W^ rows are the MFMA "A" operand).  X^_+ is not formed: X^_+ W^ = X^ W^ - X^_- W^ in exact integers, so the
// separation is three VALU instructions per dword instead of five.  After the exchange a wave owns a quarter of its half's
// half-blocks (8 accumulator registers: two runs of four columns of one row); it scales them, keeps the fp32 running sum over
// K-segments (Sec. 4.2.2 item 2; Sec. 4.3.2 last display) and stores them.
#include "seglinear_mfma_kernel.hpp"

namespace sq {

typedef float v8f __attribute__((ext_vector_type(8)));

constexpr int kKsplitSegments = 8;
struct KsplitTable {                       // the segment table of at most eight K-segments: a few cache lines of arguments
  int S;
  int kseg_off[kKsplitSegments + 1];
  int dual[kKsplitSegments];
  float s_pos[kKsplitSegments];
  float s_neg[kKsplitSegments];
};

template <int BM, int BN, int WM, int WN, bool DUAL>
struct KsplitCfg {
  static constexpr int KW = 4;                                     // waves that share a part of the tile and split K
  static constexpr int NW = WM * WN * KW;
  static constexpr int IM = BM / WM / 32, JN = BN / WN / 32;       // 32x32 blocks of a wave
  static constexpr int STAGE = (BM + BN) * 128;
  static constexpr int GA = BM / 8 / NW;                           // direct loads of a wave and stage: X^ rows ...
  static constexpr int GB = BN / 8 / NW;                           // ... and W^ rows
  static constexpr int NU = 2 * IM * JN, UPW = NU / KW;            // half-blocks of a wave's part, and of its owner's share
  static constexpr int POL = DUAL ? 2 : 1;
  static constexpr int XPHASE = NW * KW * POL * 2048;              // exchange: one half-block per owner, all waves
  static constexpr int RAW = 144 * 1024 / STAGE;
  static constexpr int NS = RAW > 9 ? 9 : RAW;
  static constexpr int LDS = NS * STAGE > XPHASE ? NS * STAGE : XPHASE;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && NU % KW == 0, "tile");
  static_assert(NS >= 3 && LDS <= 160 * 1024, "LDS budget");
};

template <int BM, int BN, int WM, int WN, bool DUAL, bool MULTI>
__global__ __launch_bounds__(WM * WN * 256, 2) void seglinear_ksplit_kernel(const GemmArgs a, const KsplitTable tb, const int mode) {
  using C = KsplitCfg<BM, BN, WM, WN, DUAL>;
  constexpr int IM = C::IM, JN = C::JN, GA = C::GA, GB = C::GB, NS = C::NS, STAGE = C::STAGE, NW = C::NW, NU = C::NU, UPW = C::UPW;
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kw = wave & 3, part = wave >> 2;
  const int wm = part / WN, wn = part % WN;

  // the workgroup's tile (one each, the grid is the tile list): each XCD (workgroup ids are dealt round-robin) takes a contiguous run
  // of the list, ordered in panels of group_m row tiles, so that the tiles on an XCD share operand rows in its L2
  const int ntiles = a.tiles_m * a.tiles_n;
  const int xcd = blockIdx.x & 7, xper = ntiles >> 3, xrem = ntiles & 7;
  const int logical = (xcd < xrem ? xcd * (xper + 1) : xrem * (xper + 1) + (xcd - xrem) * xper) + (blockIdx.x >> 3);
  const int gsz = a.group_m * a.tiles_n, g = logical / gsz, in = logical - g * gsz, first = g * a.group_m;
  const int gm = (a.tiles_m - first) < a.group_m ? (a.tiles_m - first) : a.group_m;
  const int tn = in / gm;
  const int m0 = (first + (in - tn * gm)) * BM, n0 = tn * BN;

  const uint32_t lds0 = (uint32_t)(uintptr_t)SQ_LDS(smem);
  const int lrow = lane >> 3, lslot = lane & 7;
  constexpr int NL = GA + GB;                                      // direct loads of a wave per stage
  const int frow = lane & 31;
  const int foff = frow * 128 + (((2 * kw + (lane >> 5)) ^ row_swizzle<128>(frow)) << 4);
  const char* fragA = smem + wm * (IM * 32 * 128) + foff;
  const char* fragB = smem + BM * 128 + wn * (JN * 32 * 128) + foff;
  // Constants and results travel in pieces of column_of(), at any alignment (value by value where a row was ragged or N no multiple
  // of eight: 333 x 6144 x 1535 22.1 us with its quantizer, 20.8 now; 512 x 12288 x 3071 50.5, 47.4).
  const bool pieces = a.N >= 8;
  typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
  typedef int v4iu __attribute__((ext_vector_type(4), aligned(2)));

  uint32_t voffA[GA], voffB[GB];
#pragma unroll
  for (int e = 0; e < GA; ++e) {
    const int rt = (e * NW + wave) * 8 + lrow;
    int r = m0 + rt;
    r = r < a.M ? r : a.M - 1;                                   // ragged tail: re-read the last row, masked at the store
    voffA[e] = (uint32_t)r * (uint32_t)a.K + (uint32_t)((lslot ^ row_swizzle<128>(rt)) << 4);
  }
#pragma unroll
  for (int e = 0; e < GB; ++e) {
    const int rt = (e * NW + wave) * 8 + lrow;
    const int r = column_of(n0, rt, a.N);
    voffB[e] = (uint32_t)r * (uint32_t)a.K + (uint32_t)((lslot ^ row_swizzle<128>(rt)) << 4);
  }

  v8f fsum[MULTI ? UPW : 1];
#pragma unroll
  for (int u = 0; u < (MULTI ? UPW : 1); ++u) fsum[u] = (v8f)(0.0f);

#pragma unroll 1
  for (int ks = 0; ks < (MULTI ? tb.S : 1); ++ks) {
    const int kbeg = MULTI ? tb.kseg_off[ks] : 0, n = ((MULTI ? tb.kseg_off[ks + 1] : a.K) - kbeg) >> 7;   // stages of the segment
    const bool dl = DUAL && (!MULTI || tb.dual[ks] != 0);
    const int8_t* xbase = a.xq + kbeg;
    const int8_t* wbase = a.wq + kbeg;
    auto uniform_ptr = [](const int8_t* p) __attribute__((always_inline)) {
      const uint64_t u = reinterpret_cast<uint64_t>(p);
      const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
      return reinterpret_cast<const int8_t*>(((uint64_t)hi << 32) | lo);
    };
    int islot = 0, rslot = 0;                                    // ring slots of the next stage to fetch / to read
    const int8_t *pa = xbase, *pb = wbase;                       // operand bases of the next stage to fetch
    uint32_t so = 0;
    auto issue_begin = [&]() __attribute__((always_inline)) {
      so = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)islot * (uint32_t)STAGE + (uint32_t)wave * 1024u);
      pa = uniform_ptr(pa);
      pb = uniform_ptr(pb);
    };
    auto issue_load = [&](const int e) __attribute__((always_inline)) {   // e is a compile-time constant after unrolling
      if (e < GA) {
        glds16(pa, voffA[e < GA ? e : 0], so + (uint32_t)(e * NW) * 1024u);
      } else {
        const int g = e - GA;
        glds16(pb, voffB[g >= 0 ? g : 0], so + (uint32_t)(BM / 8 + g * NW) * 1024u);
      }
    };
    auto issue_end = [&]() __attribute__((always_inline)) {
      islot = (islot + 1 == NS) ? 0 : islot + 1;
      pa += 128;
      pb += 128;
    };
    // all loads of this wave up to a stage have landed when at most `after` later stages are outstanding
    auto wait_after = [&](const int after) __attribute__((always_inline)) {
      const int left = after * NL;
      if (left >= 12) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
      else if (left >= 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
      else if (left >= 3) asm volatile("s_waitcnt vmcnt(3)" ::: "memory");
      else if (left >= 2) asm volatile("s_waitcnt vmcnt(2)" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };

    v16i accp[IM][JN], accn[DUAL ? IM : 1][DUAL ? JN : 1];
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) {
        accp[i][j] = (v16i)(0);
        if (DUAL) accn[i][j] = (v16i)(0);
      }
    v4i ap[2][IM], an[2][DUAL ? IM : 1], bf[JN - 1], bl[2];     // bl: the last block column, two sets

    // The MFMAs of one stage (set c), one per slot, interleaved with the fragment reads of the next stage, (DL) their
    // polarity separation and the direct loads of stage s + NS.  Block column by block column, so that a column's W^
    // fragment register is refilled right behind its last use; the last column has two sets, so that no read is young at
    // the barrier.
    auto iter = [&](auto dl_tag, auto c_tag, auto pf_tag, auto more_tag, const int s) __attribute__((always_inline)) {
      constexpr bool DL = decltype(dl_tag)::value;
      constexpr bool PF = decltype(pf_tag)::value;
      constexpr int c = decltype(c_tag)::value, NP = DL ? 2 : 1, NM = IM * JN * NP;
      constexpr int QV_RAW = IM + 2, QV0 = QV_RAW < NM - 1 ? QV_RAW : NM - 1;        // first slot with separation work
      constexpr int ND = DL ? IM * 4 : 0, DPS = ND ? (ND + NM - QV0 - 1) / (NM - QV0) : 0;
      constexpr bool ALWAYS = decltype(more_tag)::value;         // there are stages left to fetch: the steady state
      const bool more = PF && (ALWAYS || s + NS < n);
      if (PF) {
        if (ALWAYS) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * NL) : "memory");
        else wait_after((s + NS < n ? s + NS : n) - (s + 2));
        __syncthreads();                                         // stage s + 1 is published, stage s is read by everybody
        rslot = (rslot + 1 == NS) ? 0 : rslot + 1;
        issue_begin();
      }
      const char* fa = fragA + rslot * STAGE;
      const char* fb = fragB + rslot * STAGE;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int j = q / (IM * NP), i = (q / NP) % IM;
        const v4i bv = j + 1 < JN ? bf[j + 1 < JN ? j : 0] : bl[c];
        if (NP == 1 || q % NP == 0) accp[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bv, ap[c][i], accp[i][j], 0, 0, 0);
        else accn[DUAL ? i : 0][DUAL ? j : 0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bv, an[c][DUAL ? i : 0], accn[DUAL ? i : 0][DUAL ? j : 0], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (PF) {
          if (q < IM) ap[c ^ 1][q < IM ? q : 0] = *reinterpret_cast<const v4i*>(fa + (q < IM ? q : 0) * (32 * 128));
          if (q == (IM < NM ? IM - 1 : 0)) bl[c ^ 1] = *reinterpret_cast<const v4i*>(fb + (JN - 1) * (32 * 128));
          if (j + 1 < JN && q % (IM * NP) == IM * NP - 1) bf[j + 1 < JN ? j : 0] = *reinterpret_cast<const v4i*>(fb + j * (32 * 128));
          if (ND && q >= QV0) {
#pragma unroll
            for (int d = 0; d < DPS; ++d) {
              const int w = (q - QV0) * DPS + d;
              if (w < ND) {
                int neg = negative_codes(ap[c ^ 1][w / 4][w % 4]);
                asm volatile("" : "+v"(neg));                    // done here, not sunk behind the next barrier
                an[c ^ 1][DUAL ? w / 4 : 0][w % 4] = neg;
              }
            }
          }
#pragma unroll
          for (int e = 0; e < NL; ++e) {                         // spread over the slots behind the X^ reads
            constexpr int Q0 = IM < NM ? IM : NM - 1;
            if (Q0 + e * (NM - Q0) / NL == q && more) issue_load(e);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) issue_end();
    };
    auto k_loop = [&](auto dl_tag) __attribute__((always_inline)) {
      constexpr bool DL = decltype(dl_tag)::value;
      std::integral_constant<int, 0> c0;
      std::integral_constant<int, 1> c1;
      const int np = n < NS ? n : NS;
#pragma unroll 1
      for (int s = 0; s < np; ++s) {
        issue_begin();
#pragma unroll
        for (int e = 0; e < GA + GB; ++e) issue_load(e);
        issue_end();
      }
      wait_after(np - 1);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < IM; ++i) ap[0][i] = *reinterpret_cast<const v4i*>(fragA + i * (32 * 128));
#pragma unroll
      for (int j = 0; j + 1 < JN; ++j) bf[j] = *reinterpret_cast<const v4i*>(fragB + j * (32 * 128));
      bl[0] = *reinterpret_cast<const v4i*>(fragB + (JN - 1) * (32 * 128));
      if (DL) {
#pragma unroll
        for (int i = 0; i < IM; ++i)
#pragma unroll
          for (int d = 0; d < 4; ++d) an[0][DUAL ? i : 0][d] = negative_codes(ap[0][i][d]);
      }
      std::true_type yes;
      std::false_type no;
      int s = 0;
      // an odd number of stages is left for the loops below, so that every K loop ends on one copy of the last iteration
      // (two copies that meet behind the loop cost the register allocator a second accumulator set)
      if ((n & 1) == 0) {
        iter(dl_tag, c0, yes, no, 0);
#pragma unroll
        for (int i = 0; i < IM; ++i) {
          ap[0][i] = ap[1][i];
          if (DL) an[0][DUAL ? i : 0] = an[1][DUAL ? i : 0];
        }
        bl[0] = bl[1];
        s = 1;
      }
#pragma unroll 1
      for (; s + 1 + NS < n; s += 2) {
        iter(dl_tag, c0, yes, yes, s);
        iter(dl_tag, c1, yes, yes, s + 1);
      }
#pragma unroll 1
      for (; s + 1 < n; s += 2) {
        iter(dl_tag, c0, yes, no, s);
        iter(dl_tag, c1, yes, no, s + 1);
      }
      iter(dl_tag, c0, no, no, s);
    };
    if (dl) k_loop(std::integral_constant<bool, DUAL>{});
    else k_loop(std::false_type{});

    // ---- exchange and flush: in phase w the waves of a part hand half-block w of every owner over, who adds, scales and
    // (last K-segment) stores.  One body for all phases: unrolled, the owners' sums of several phases are live next to the
    // accumulators.
    const bool last = !MULTI || ks + 1 == tb.S;
#pragma unroll 1
    for (int w = 0; w < UPW; ++w) {
      const int u = kw * UPW + w, b = u >> 1, p = u & 1, i = b / JN, j = b - i * JN;
      const int nb = n0 + (wn * JN + j) * 32 + 16 * p;           // the half-block's 16 columns
      const int m = m0 + (wm * IM + i) * 32 + frow;
      const int np[2] = {piece_of(nb, a.N), piece_of(nb + 8, a.N)};
      const int nc[2] = {np[0] + 4 * (lane >> 5), np[1] + 4 * (lane >> 5)};   // this lane's columns: four from each on
      const bool in_m = m < a.M;
      // the constants are requested in front of the exchange, which covers their latency (the raw-sum mode has none: its
      // caller passes no wscale)
      float sp = tb.s_pos[MULTI ? ks : 0], sn = dl ? tb.s_neg[MULTI ? ks : 0] : 0.0f;
      if (a.tok_steps) {                                         // dynamic per-token steps of this lane's row
        const int mr = in_m ? m : a.M - 1;
        sp = a.tok_steps[(size_t)mr * tb.S + ks];
        sn = dl ? a.tok_steps[((size_t)a.M + mr) * tb.S + ks] : 0.0f;
      }
      const bool add_bias = last && a.bias != nullptr;
      float cw[8] = {}, bs[8] = {};
      if (mode != OUT_DEBUG_ACC) {
        const float* ws = a.wscale + (size_t)ks * a.N;
        const float* bias = add_bias ? a.bias : ws;
        if (pieces) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const v4f w4 = *reinterpret_cast<const v4fu*>(ws + nc[h]), b4 = *reinterpret_cast<const v4fu*>(bias + nc[h]);
#pragma unroll
            for (int r = 0; r < 4; ++r) { cw[4 * h + r] = w4[r]; bs[4 * h + r] = b4[r]; }
          }
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const int n = nc[r >> 2] + (r & 3), nv = n < a.N ? n : a.N - 1;
            cw[r] = ws[nv];
            bs[r] = bias[nv];
          }
        }
      }
      __syncthreads();                                           // the ring (or the previous phase) has been read
      char* to = smem + wave * (C::KW * C::POL * 2048) + lane * 16;
#pragma unroll
      for (int ws_ = 0; ws_ < UPW; ++ws_)
        if (w == ws_) {
#pragma unroll
          for (int o = 0; o < C::KW; ++o) {
            const int uo = o * UPW + ws_, io = (uo >> 1) / JN, jo = (uo >> 1) % JN, po = uo & 1;
#pragma unroll
            for (int h = 0; h < C::POL; ++h) {
              v16i& v = h == 0 ? accp[io][jo] : accn[DUAL ? io : 0][DUAL ? jo : 0];
              *reinterpret_cast<v4i*>(to + (o * C::POL + h) * 2048) = (v4i){v[8 * po], v[8 * po + 1], v[8 * po + 2], v[8 * po + 3]};
              *reinterpret_cast<v4i*>(to + (o * C::POL + h) * 2048 + 1024) = (v4i){v[8 * po + 4], v[8 * po + 5], v[8 * po + 6], v[8 * po + 7]};
            }
          }
        }
      __syncthreads();
      v8i sum[C::POL];                                           // X^ W^ (and X^_- W^) of the whole segment
#pragma unroll
      for (int src = 0; src < C::KW; ++src)
#pragma unroll
        for (int h = 0; h < C::POL; ++h) {
          const char* from = smem + (part * C::KW + src) * (C::KW * C::POL * 2048) + (kw * C::POL + h) * 2048 + lane * 16;
          const v4i lo = *reinterpret_cast<const v4i*>(from), hi = *reinterpret_cast<const v4i*>(from + 1024);
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            sum[h][d] = src == 0 ? lo[d] : sum[h][d] + lo[d];
            sum[h][4 + d] = src == 0 ? hi[d] : sum[h][4 + d] + hi[d];
          }
        }
      if (DUAL && dl) sum[0] -= sum[C::POL - 1];                 // X^_+ W^ = X^ W^ - X^_- W^, exactly
      if (mode == OUT_DEBUG_ACC) {
        if (in_m) {
          const size_t o = ((size_t)ks * a.M + m) * a.N;
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const int n = nc[r >> 2] + (r & 3);
            if (n < a.N) {
              a.acc_pos[o + n] = sum[0][r];
              a.acc_neg[o + n] = dl ? sum[C::POL - 1][r] : 0;
            }
          }
        }
        continue;
      }
      v8f fs = fsum[0];                                          // running sum of the earlier K-segments
#pragma unroll
      for (int q = 1; q < (MULTI ? UPW : 1); ++q) fs = w == q ? fsum[MULTI ? q : 0] : fs;
      float tv[8];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        float v = (cw[r] * sp) * (float)sum[0][r];
        if (DUAL) v += (cw[r] * sn) * (dl ? (float)sum[C::POL - 1][r] : 0.0f);
        if (MULTI) v += fs[r];
        tv[r] = v;
      }
      if (!last) {
#pragma unroll
        for (int q = 0; q < UPW; ++q)
          if (w == q)
#pragma unroll
            for (int r = 0; r < 8; ++r) fsum[MULTI ? q : 0][r] = tv[r];
        continue;
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) tv[r] += add_bias ? bs[r] : 0.0f;
      const size_t o = (size_t)m * a.N;
      if (mode == OUT_BF16) {
        uint16_t* y = reinterpret_cast<uint16_t*>(a.y);
        if (pieces) {
          const uint32_t a0 = f32x2_to_bf16x2(tv[0], tv[1]), a1 = f32x2_to_bf16x2(tv[2], tv[3]);
          const uint32_t b0 = f32x2_to_bf16x2(tv[4], tv[5]), b1 = f32x2_to_bf16x2(tv[6], tv[7]);
          // lanes 32..63 of the first operand <-> lanes 0..31 of the second: a piece per lane
          const auto s0 = __builtin_amdgcn_permlane32_swap(a0, b0, false, false);
          const auto s1 = __builtin_amdgcn_permlane32_swap(a1, b1, false, false);
          if (in_m) *reinterpret_cast<v4iu*>(y + o + (lane < 32 ? np[0] : np[1])) = (v4iu){(int)s0[0], (int)s1[0], (int)s0[1], (int)s1[1]};
        } else if (in_m) {
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const int n = nc[r >> 2] + (r & 3);
            if (n < a.N) y[o + n] = f32_to_bf16(tv[r]);
          }
        }
      } else if (in_m) {
        float* y = reinterpret_cast<float*>(a.y);
        if (pieces) {
          *reinterpret_cast<v4fu*>(y + o + nc[0]) = (v4fu){tv[0], tv[1], tv[2], tv[3]};
          *reinterpret_cast<v4fu*>(y + o + nc[1]) = (v4fu){tv[4], tv[5], tv[6], tv[7]};
        } else {
#pragma unroll
          for (int r = 0; r < 8; ++r) {
            const int n = nc[r >> 2] + (r & 3);
            if (n < a.N) y[o + n] = tv[r];
          }
        }
      }
    }
    // the next segment counts its direct loads from zero and overwrites the exchange area
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }
}

template <int BM, int BN, int WM, int WN>
static hipError_t launch_cfg(const GemmArgs& a, const KsplitTable& tb, int mode, bool dual, int grid, hipStream_t st) {
#define SQ_K(D, MS) hipLaunchKernelGGL((seglinear_ksplit_kernel<BM, BN, WM, WN, D, MS>), dim3(grid), dim3(WM * WN * 256), 0, st, a, tb, mode)
  if (tb.S > 1) { if (dual) SQ_K(true, true); else SQ_K(false, true); }
  else { if (dual) SQ_K(true, false); else SQ_K(false, false); }
#undef SQ_K
  return hipGetLastError();
}

struct KsplitTile { int BM, BN; };
static const KsplitTile kTiles[3] = {{64, 64}, {64, 128}, {128, 64}};
static long tile_count(const GemmArgs& a, int t) {
  return (long)((a.M + kTiles[t].BM - 1) / kTiles[t].BM) * ((a.N + kTiles[t].BN - 1) / kTiles[t].BN);
}

bool ksplit_supported(const GemmArgs& a, const GemmTable& tb) {
  if (tb.S > kKsplitSegments || tb.has_seg_scale) return false;
  for (int s = 0; s <= tb.S; ++s)
    if (tb.kseg_off[s] % 128 != 0) return false;
  return (reinterpret_cast<uintptr_t>(a.xq) | reinterpret_cast<uintptr_t>(a.wq)) % 16 == 0;
}

// The tile, or -1 where the tile kernel serves: the layer has more tiles than there are compute units, or its K-segments are too
// short for it.  A second round of tiles repeats the exposed start and exchange (3 - 7 us; the tile kernel fetches across tiles)
// and made this kernel the slower one on all but one of 16 layers (1296 x 8192 x 2048: 61 against 55 us).  A K-segment costs a
// start, a drain and an exchange (0.3 - 0.5 us on the tiles with 64 columns, 2 us on 64 x 128), which its stages of 128 columns have
// to earn back: about 0.2 us each where both polarity paths run, 0.07 where one does (64 x 128: 0.09 and 0.02).  The lines were
// drawn with the tile kernel as it was when none of 1039 layers taken lost more than 1.5 %.  Against the present one, 777 layers taken (1 - 8
// segments of 128 - 12288 columns, 33 - 20000 rows, every mix of paths): one segment on 64 x 64 tiles 0.71 of its time in the median and
// never more than 0.94; several there 0.92, 63 of 526 more than 1.02, 1.14 at the most; on 64 x 128 tiles one 0.99, several (18 layers) 1.05 - 1.25
// (2193 x 640, four of 5248 columns, two of them with both paths: 67.3 us there, 83.8 here).  Many short segments, which are not taken, took up
// to 2.3 times as long (522 x 2112, eight of 128: 15.5 us there, 35.4 here).
// One segment on 64 x 128 tiles, ten shapes, when the lines were drawn: 2048 columns of one path took 0.95 - 0.81 of the tile kernel's time, 1536 of them
// 1.03 - 0.87; 2304 of two paths 0.97 - 0.81, 2048 of them 1.03 - 0.89, 1536 of them up to 1.25.
int ksplit_pick(const GemmArgs& a, const GemmTable& tb) {
  if (!ksplit_supported(a, tb)) return -1;
  int tile = 0;
  while (tile < 3 && tile_count(a, tile) > device_cus()) ++tile;
  if (tile == 3) return -1;
  const int S = tb.S;
  int both = 0, one = 0;                                           // stages in segments with two paths / with one
  for (int s = 0; s < S; ++s) (tb.dual[s] ? both : one) += (tb.kseg_off[s + 1] - tb.kseg_off[s]) >> 7;
  bool earns;
  if (tile == 1) {
    earns = S == 1 ? both >= 18 || one >= 16 : both > 0 && 6 * both + one >= 128 * S + 16;
  } else if (both == 0) {
    earns = tile == 2 ? S <= 2 : (S <= 3 || one >= 24 * S);
  } else if (one == 0) {
    earns = S <= 4 || both >= 2 * S;
  } else {
    earns = both + one >= 2 * S && 5 * both >= 2 * one + 12;
  }
  return earns ? tile : -1;
}

hipError_t launch_seglinear_ksplit(GemmArgs a, const GemmTable& tb, OutMode mode, int tile, hipStream_t st) {
  if (tile < 0 || tile >= 3 || !ksplit_supported(a, tb)) return hipErrorInvalidConfiguration;
  KsplitTable kt{};
  kt.S = tb.S;
  bool dual = false;
  for (int s = 0; s < tb.S; ++s) {
    kt.kseg_off[s + 1] = tb.kseg_off[s + 1];
    kt.dual[s] = tb.dual[s];
    kt.s_pos[s] = tb.s_pos[s];
    kt.s_neg[s] = tb.s_neg[s];
    dual = dual || tb.dual[s] != 0;
  }
  a.tiles_m = (a.M + kTiles[tile].BM - 1) / kTiles[tile].BM;
  a.tiles_n = (a.N + kTiles[tile].BN - 1) / kTiles[tile].BN;
  a.group_m = a.tiles_m < 8 ? a.tiles_m : 8;
  const int grid = a.tiles_m * a.tiles_n;
  if (tile == 0) return launch_cfg<64, 64, 2, 1>(a, kt, mode, dual, grid, st);
  if (tile == 1) return launch_cfg<64, 128, 1, 2>(a, kt, mode, dual, grid, st);
  return launch_cfg<128, 64, 2, 1>(a, kt, mode, dual, grid, st);
}

}  // namespace sq
