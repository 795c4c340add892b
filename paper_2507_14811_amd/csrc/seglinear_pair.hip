// SegLinear GEMM for large layers of one K-segment without a polarity split (Sec. 4.2.2), int8 or E4M3 codes.
//
// The kernel of seglinear_mfma_kernel.hpp has one wave per SIMD: while it scales, converts and stores a tile the matrix cores
// idle (a fifth of the time at K = 1536), and the loads of its next K loop complete behind the stores.  A layer without a polarity
// split needs one accumulator set, half of the registers, so here two groups of four waves share a compute unit and take its tiles
// in turn: one group runs the K loop of its tile while the other one stores its last tile, a few rows of each 32 x 32 block between two
// barriers.  Both groups pass the same barriers, one per 128-byte stage.
//   * The group in its K loop fetches (direct global->LDS loads, ring of three stages across all tiles), so its loads do not wait
//     behind the stores of the other group.  Its own stores have the rest of that group's K loop and two stages of its next one
//     until a wait counts them: little with K = 512, where they take three of the four stages.  Shared between the groups instead,
//     the loads waited behind stores (4608 x 3072 x 12288 with bf16 output 154 -> 147 us, 8500 x 1536 x 4608 59 -> 56, zero codes).
//   * wscale, bias and token steps of a tile come by direct loads into LDS at the start of its K loop, so the store code has no
//     memory latency of its own.
//   * X^ rows are the MFMA "A" operand (the other way round than in the tile kernel), and W^ rows lie in a stage in the order that gives a
//     lane BN / 64 neighbouring columns of a row: it stores what it holds, one row piece of 32 lanes x BN / 64 columns beside the next,
//     at any alignment, and has one scale and bias per column instead of sixteen per block.  A 32 x 32
//     block at a time (64 bytes of 16 rows an instruction, behind lane swaps; odd N value by value) / this way, with the quantizer: 8500 x
//     1536 x 4608 bf16 67.6 / 65.8 us, fp32 output 103.5 / 97.5, N = 4607 121.6 / 75.0; 5500 x 896 x 2688 29.6 / 24.3; E4M3 4608 x 3072 x
//     12288 168.8 / 162.0, 4608 x 4096 x 16384 288.8 / 276.8.  Measured and not taken: of three columns two beside each other and one
//     32 further on (stores of 4 bytes a lane, lines shared between waves: 43 -> 58 us for 3000 x 2048 x 6144).
// Measured, tile kernel / here: 8500 x 1536 x 4608 bf16 74 / 64.6 us, fp32 output with token steps 93 / 74.7, E4M3 72 / 64.4;
// 4608 x 3072 x 12288 bf16 172 / 152, E4M3 167 / 149; 4733 x 896 x 3018 60 / 42.  What bounds it is the power of real codes (zero
// codes: 50 us for 8500 x 1536 x 4608), then 0.62 us per stage of a 128 x 256 tile (MFMAs 0.43, LDS reads and direct loads 0.48).
#include "seglinear_mfma_kernel.hpp"

namespace sq {

// lane l's 4 bytes land at lds_addr + 4 l
__device__ __forceinline__ void glds4(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

template <int BN, bool FP8>
struct PairCfg {
  static constexpr int BM = 128, NS = 3;
  static constexpr int IM = 2, JN = BN / 64;                       // 32x32 blocks of a wave (a group is a 2 x 2 grid of waves)
  static constexpr int STAGE = (BM + BN) * 128;
  static constexpr int GA = BM / 8 / 4, GB = BN / 8 / 4, LT = GA + GB;   // direct loads of a wave and stage
  static constexpr int FW = FP8 ? 8 : 4, CH = FW / 4, SUB = 128 / (8 * FW);
  static constexpr int CONST = (BN + BN + BM) * 4;                 // wscale, bias, token steps of a group's tile
  static constexpr int LDS = NS * STAGE + 2 * CONST;
  static_assert(BM % 32 == 0 && BN % 64 == 0 && LDS <= 160 * 1024, "tile");
  // The tile's column in place 32 (JN wn + j) + f of a stage's W^ rows: lane f of a wave holds JN neighbouring ones, one per block
  static __device__ __forceinline__ int column(int place) {
    return place / (32 * JN) * (32 * JN) + JN * (place & 31) + (place >> 5) % JN;
  }
};

template <int BN, bool TOK, bool FP8, bool BF>
__global__ __launch_bounds__(512, 2) void seglinear_pair_kernel(const GemmArgs a, const float s_pos) {
  using C = PairCfg<BN, FP8>;
  constexpr int BM = C::BM, IM = C::IM, JN = C::JN, GA = C::GA, GB = C::GB, LT = C::LT, STAGE = C::STAGE, SUB = C::SUB, CH = C::CH;
  constexpr int FW = C::FW, NB = IM * JN;                          // blocks of a wave
  using vfrag = std::conditional_t<FP8, v8i, v4i>;
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave >> 2, w4 = wave & 3, wm = w4 >> 1, wn = w4 & 1;

  // this workgroup's tiles: as in the tile kernel (a contiguous run of the panel-ordered list per XCD)
  const int ntiles = a.tiles_m * a.tiles_n;
  const int xcd = blockIdx.x & 7, xlocal = blockIdx.x >> 3;
  const int xper = ntiles >> 3, xrem = ntiles & 7;
  const int xstart = xcd < xrem ? xcd * (xper + 1) : xrem * (xper + 1) + (xcd - xrem) * xper;
  const int xcnt = xper + (xcd < xrem ? 1 : 0);
  const int xwg = (int)(gridDim.x >> 3) + (xcd < (int)(gridDim.x & 7) ? 1 : 0);
  const int ntile = xlocal < xcnt ? (xcnt - xlocal + xwg - 1) / xwg : 0;
  if (ntile == 0) return;                                          // uniform: the whole workgroup leaves
  auto tile_origin = [&](const int it, int& tm0, int& tn0) __attribute__((always_inline)) {
    const int logical = xstart + (it < ntile ? it : ntile - 1) * xwg + xlocal;
    const int gsz = a.group_m * a.tiles_n;
    const int g = logical / gsz, in = logical - g * gsz;
    const int first = g * a.group_m;
    const int gm = (a.tiles_m - first) < a.group_m ? (a.tiles_m - first) : a.group_m;
    const int tn = in / gm;
    tm0 = (first + (in - tn * gm)) * BM;
    tn0 = tn * BN;
  };
  const int nk = a.K >> 7;                                         // stages of a tile

  // ---- fetching: the waves of the group in its K loop load a quarter of every stage each ------------------------------------
  const int lrow = lane >> 3, lslot = lane & 7;
  const uint32_t lds0 = (uint32_t)(uintptr_t)SQ_LDS(smem);
  auto uniform_ptr = [](const int8_t* p) __attribute__((always_inline)) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return reinterpret_cast<const int8_t*>(((uint64_t)hi << 32) | lo);
  };
  const int8_t *fA = a.xq, *fB = a.wq;                             // operands of the stage to fetch next
  uint32_t voffA[GA], voffB[GB], iso = 0;
  auto set_fetch = [&](const int tm0, const int tn0, const int stage) __attribute__((always_inline)) {
    fA = uniform_ptr(a.xq + (size_t)tm0 * a.K + stage * 128);
    fB = uniform_ptr(a.wq + (size_t)tn0 * a.K + stage * 128);
    const int mlast = a.M - 1 - tm0, nlast = a.N - 1 - tn0;        // ragged tail: re-read the last row, masked at the store
#pragma unroll
    for (int g = 0; g < GA; ++g) {
      const int rt = (w4 * GA + g) * 8 + lrow;
      voffA[g] = (uint32_t)(rt < mlast ? rt : mlast) * (uint32_t)a.K + (uint32_t)((lslot ^ row_swizzle<128>(rt)) << 4);
    }
#pragma unroll
    for (int g = 0; g < GB; ++g) {
      const int rt = (w4 * GB + g) * 8 + lrow, col = C::column(rt);
      voffB[g] = (uint32_t)(col < nlast ? col : nlast) * (uint32_t)a.K + (uint32_t)((lslot ^ row_swizzle<128>(rt)) << 4);
    }
  };
  auto issue_load = [&](const int e) __attribute__((always_inline)) {       // e is a compile-time constant after unrolling
    if (e < GA) glds16(fA, voffA[e < GA ? e : 0], iso + (uint32_t)(w4 * GA + e) * 1024u);
    else glds16(fB, voffB[e >= GA ? e - GA : 0], iso + (uint32_t)(BM * 128) + (uint32_t)(w4 * GB + (e >= GA ? e - GA : 0)) * 1024u);
  };
  auto issue_all = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < LT; ++e) issue_load(e);
  };
  int fstep = 128;                                                 // 0 behind the last tile: its last stage is fetched again, and never read
  auto advance = [&]() __attribute__((always_inline)) {
    fA += fstep;
    fB += fstep;
  };

  // ---- the barrier of a stage: it has landed, everybody has read the one before ------------------------------------------------
  int rd = 2 * STAGE;
  auto barrier = [&]() __attribute__((always_inline)) {
    __syncthreads();
    iso = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)rd);     // the buffer of the stage before: the stage after next goes there
    rd = rd == 2 * STAGE ? 0 : rd + STAGE;
  };
  auto wait_fetched = [&]() __attribute__((always_inline)) {       // all but the loads of one stage
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LT) : "memory");
  };

  // ---- fragments and one k-step ---------------------------------------------------------------------------------------------
  const int frow = lane & 31, fsw = row_swizzle<128>(frow), fhi = lane >> 5;
  int foff[SUB];
#pragma unroll
  for (int h = 0; h < SUB; ++h) foff[h] = frow * 128 + (((2 * CH * h + CH * fhi) ^ fsw) << 4);   // E4M3: second chunk at this ^ 16
  const char* fragA = smem + (wm * IM * 32) * 128;
  const char* fragB = smem + BM * 128 + (wn * JN * 32) * 128;
  v16i acc[IM][JN];
  vfrag afr[2][IM], bfr[2][JN];
  auto read_frag = [&](const int set, const int r, const int fo) __attribute__((always_inline)) {   // read r of the IM + JN, CH pieces each
    const int f = r / CH, c = r % CH;
    const char* p = f < IM ? fragA + f * (32 * 128) : fragB + (f - IM) * (32 * 128);
    const v4i t = *reinterpret_cast<const v4i*>(p + (fo ^ (16 * c)));
    vfrag& d = f < IM ? afr[set][f < IM ? f : 0] : bfr[set][f >= IM ? f - IM : 0];
#pragma unroll
    for (int k = 0; k < 4; ++k) d[4 * c + k] = t[k];
  };
  constexpr int NR = (IM + JN) * CH;
  auto kstep = [&](auto pf_tag, auto grp_tag, const int cur, const int fo_next) __attribute__((always_inline)) {
    constexpr bool PF = decltype(pf_tag)::value;
    constexpr int GRP = decltype(grp_tag)::value;
    constexpr int RPS = (NR + NB - 1) / NB;                        // LDS reads per MFMA
    constexpr int NG = GRP >= 0 ? ((GRP + 1) * LT + SUB - 1) / SUB - (GRP * LT + SUB - 1) / SUB : 0;
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int i = q / JN, j = q % JN;
      if constexpr (FP8) {
        acc[i][j] = __builtin_bit_cast(v16i, __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
            afr[cur][i], bfr[cur][j], __builtin_bit_cast(v16f, acc[i][j]), 0, 0, 0, 0, 0, 0));
      } else {
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(afr[cur][i], bfr[cur][j], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (PF) {
#pragma unroll
        for (int r = 0; r < NR; ++r)
          if (r / RPS == q) read_frag(cur ^ 1, r, fo_next);
      }
      if (GRP >= 0) {
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < LT; ++e)
          if (e * SUB / LT == GRP) {
            if (NB - NG + cnt == q) issue_load(e);                 // behind the reads
            ++cnt;
          }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto first_steps = [&](auto fetch_tag) __attribute__((always_inline)) {    // k-steps 0 .. SUB-2 of the stage at rd
    constexpr bool F = decltype(fetch_tag)::value;
#pragma unroll
    for (int h = 0; h + 1 < SUB; ++h) {
      if (h == 0) kstep(std::true_type{}, std::integral_constant<int, F ? 1 : -1>{}, 0, rd + foff[1]);
      if (h == 1) kstep(std::true_type{}, std::integral_constant<int, F ? 2 : -1>{}, 1, rd + foff[SUB > 2 ? 2 : 0]);
      if (h == 2) kstep(std::true_type{}, std::integral_constant<int, F ? 3 : -1>{}, 0, rd + foff[SUB > 3 ? 3 : 0]);
    }
  };
  constexpr int LASTSET = (SUB - 1) & 1;
  auto stage_slot = [&]() __attribute__((always_inline)) {                   // last k-step of the stage before, then this stage's
    kstep(std::true_type{}, std::integral_constant<int, 0>{}, LASTSET, rd + foff[0]);
    first_steps(std::true_type{});
    advance();
  };

  // ---- constants of the group's tile: by direct loads into LDS, so that the store code has no load of its own to wait for -----
  const uint32_t ldsC = lds0 + (uint32_t)(C::NS * STAGE + group * C::CONST);
  const float* cst = reinterpret_cast<const float*>(smem + C::NS * STAGE + group * C::CONST);
  const bool has_bias = a.bias != nullptr;
  int m0 = 0, n0 = 0;                                              // the group's tile
  auto fetch_constants = [&]() __attribute__((always_inline)) {
    int n = n0 + w4 * 64 + lane;
    n = n < a.N ? n : a.N - 1;
    if (w4 * 64 < BN) {
      glds4(a.wscale, (uint32_t)n * 4u, ldsC + (uint32_t)w4 * 256u);
      if (has_bias) {
        glds4(a.bias, (uint32_t)n * 4u, ldsC + (uint32_t)(BN * 4) + (uint32_t)w4 * 256u);
      }
    }
    if (TOK && w4 < 2) {
      int m = m0 + w4 * 64 + lane;
      m = m < a.M ? m : a.M - 1;
      glds4(a.tok_steps, (uint32_t)m * 4u, ldsC + (uint32_t)(2 * BN * 4) + (uint32_t)w4 * 256u);
    }
  };

  // ---- a run of four rows: scale, add the bias, store ---------------------------------------------------------------------------
  // Element v of block (i, j) in lane l: row 8 (v >> 2) + 4 (l >> 5) + (v & 3), and column f = l % 32 of the block's places.  Stored as
  // it lies: JN neighbouring columns of a row per lane, so that a store instruction covers JN x 32 consecutive columns of two rows.
  // bf16: neighbouring lanes exchange a row of every two, for twice as many columns of a row per lane.
  float cw[JN], bs[JN];
  auto tile_constants = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const int col = C::column((wn * JN + j) * 32 + frow);
      cw[j] = TOK ? cst[col] : cst[col] * s_pos;
      bs[j] = has_bias ? cst[BN + col] : 0.0f;
    }
  };
  auto store_run = [&](auto full_tag, const int i, const int g) __attribute__((always_inline)) {
    constexpr bool FULL = decltype(full_tag)::value;
    const int row = (wm * IM + i) * 32 + 8 * g + 4 * fhi;
    const int m = m0 + row, n = n0 + 32 * JN * wn + JN * frow;
    v4f sp = (v4f)(1.0f);
    if (TOK) sp = *reinterpret_cast<const v4f*>(cst + 2 * BN + row);
    float d[4][JN];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < JN; ++j) d[r][j] = (TOK ? cw[j] * sp[r] : cw[j]) * acc_value<FP8>(acc[i][j][4 * g + r]) + bs[j];
    if constexpr (BF) {
      typedef int vst __attribute__((ext_vector_type(JN), aligned(2)));   // rows of any N
      const bool odd = (lane & 1) != 0;
      auto swap = [](const int v) __attribute__((always_inline)) { return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false); };   // lane ^ 1
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const int mm = m + r + (odd ? 1 : 0), nn = n - (odd ? JN : 0);    // this lane's row, and 2 JN columns of it
        vst o;
        if constexpr (JN == 3) {
          float t[6];
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const float got = __int_as_float(swap(__float_as_int(odd ? d[r][j] : d[r + 1][j])));
            t[j] = odd ? got : d[r][j];
            t[3 + j] = odd ? d[r + 1][j] : got;
          }
#pragma unroll
          for (int k = 0; k < 3; ++k) o[k] = (int)f32x2_to_bf16x2(t[2 * k], t[2 * k + 1]);
        } else {
#pragma unroll
          for (int k = 0; k < JN / 2; ++k) {
            const int p0 = (int)f32x2_to_bf16x2(d[r][2 * k], d[r][2 * k + 1]), p1 = (int)f32x2_to_bf16x2(d[r + 1][2 * k], d[r + 1][2 * k + 1]);
            const int got = swap(odd ? p0 : p1);
            o[k] = odd ? got : p0;
            o[JN / 2 + k] = odd ? p1 : got;
          }
        }
        uint16_t* to = reinterpret_cast<uint16_t*>(a.y) + (size_t)mm * a.N + nn;
        if (FULL || (mm < a.M && nn + 2 * JN <= a.N)) {
          *reinterpret_cast<vst*>(to) = o;
        } else if (mm < a.M) {
#pragma unroll
          for (int k = 0; k < 2 * JN; ++k)
            if (nn + k < a.N) to[k] = (uint16_t)((uint32_t)o[k >> 1] >> (16 * (k & 1)));
        }
      }
    } else {
      typedef float vst __attribute__((ext_vector_type(JN), aligned(4)));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float* to = reinterpret_cast<float*>(a.y) + (size_t)(m + r) * a.N + n;
        if (FULL || (m + r < a.M && n + JN <= a.N)) {
          vst t;
#pragma unroll
          for (int j = 0; j < JN; ++j) t[j] = d[r][j];
          *reinterpret_cast<vst*>(to) = t;
        } else if (m + r < a.M) {
#pragma unroll
          for (int j = 0; j < JN; ++j)
            if (n + j < a.N) to[j] = d[r][j];
        }
      }
    }
  };

  // ---- the program of a wave: [an idle turn of group 1,] then K loop and stores of every second tile ---------------------------
  int om0, on0, nm0 = 0, nn0 = 0;                                  // origins of the group's next tile and of the one behind it
  tile_origin(group, om0, on0);
  tile_origin(group + 1, nm0, nn0);
  if (group == 0) {
    set_fetch(om0, on0, 0);
#pragma unroll
    for (int s = 0; s < C::NS; ++s) {
      iso = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(s * STAGE));
      issue_all();
      advance();
    }
  } else {
    set_fetch(om0, on0, 2);
#pragma unroll 1
    for (int i = 0; i < nk; ++i) barrier();
  }
  constexpr int NRUN = 4 * IM;                                     // runs of a tile to store
  const int per_slot = (NRUN + nk - 2) / (nk - 1);                 // of them between two barriers
#pragma unroll 1
  for (int t = group; t < ntile; t += 2) {
    m0 = om0;
    n0 = on0;
    // K loop
    __builtin_amdgcn_s_setprio(2);
#pragma unroll
    for (int h = 0; h < SUB; ++h) asm volatile("" : "+v"(foff[h]));
#pragma unroll
    for (int g = 0; g < GA; ++g) asm volatile("" : "+v"(voffA[g]));
#pragma unroll
    for (int g = 0; g < GB; ++g) asm volatile("" : "+v"(voffB[g]));
    if (t == 0) wait_fetched();                                    // later tiles: the other group fetched the first two stages
    barrier();
    if (t > 0) {
      issue_all();
      advance();
    }
    fetch_constants();
#pragma unroll
    for (int r = 0; r < NR; ++r) read_frag(0, r, rd + foff[0]);
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[i][j] = (v16i)(0);
    first_steps(std::false_type{});
    int i = 1;
#pragma unroll 1
    for (; i < nk - 2; ++i) {
      if (i > 1 || t == 0) wait_fetched();
      barrier();
      stage_slot();
    }
    if (t + 1 < ntile) set_fetch(nm0, nn0, 0);
    else { fstep = 0; fA -= 128; fB -= 128; }
#pragma unroll 1
    for (; i < nk; ++i) {
      wait_fetched();
      barrier();
      stage_slot();
    }
    // stores, next to the other group's K loop (if it has another tile): first the next tile's first two stages, which this
    // group has fetched, then run by run
    __builtin_amdgcn_s_setprio(0);
    const bool beside = t + 1 < ntile;
    if (beside) {
      wait_fetched();
      barrier();
    }
    kstep(std::false_type{}, std::integral_constant<int, -1>{}, LASTSET, 0);
    if (beside) {
      tile_origin(t + 2, om0, on0);
      tile_origin(t + 3, nm0, nn0);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    tile_constants();
    const bool full = m0 + BM <= a.M && n0 + BN <= a.N;
    int slots = 1, left = 0;
#pragma unroll
    for (int b = 0; b < NRUN; ++b) {
      if (left == 0) {
        left = per_slot;
        if (beside) {
          barrier();
          ++slots;
        }
      }
      --left;
      if (full) store_run(std::true_type{}, b >> 2, b & 3);
      else store_run(std::false_type{}, b >> 2, b & 3);
    }
    if (beside) {
      set_fetch(om0, on0, 2);
#pragma unroll 1
      for (; slots < nk; ++slots) barrier();
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // no direct load outlives its workgroup's LDS
}

bool pair_supported(const GemmArgs& a, const GemmTable& tb, OutMode mode, int tile, bool fp8) {
  return tile >= (fp8 ? 1 : 0) && tile < 3 && mode != OUT_DEBUG_ACC && tb.S == 1 && !tb.dual[0] && !tb.has_seg_scale && a.K % 128 == 0 &&
         a.K >= 512 && (reinterpret_cast<uintptr_t>(a.xq) | reinterpret_cast<uintptr_t>(a.wq)) % 16 == 0 && !(fp8 && a.tok_steps != nullptr);
}

// The tile (0: 128 x 256, 1: 128 x 192, 2: 128 x 128), or -1 where the tile kernel serves.  Among the tiles the one with the
// shortest time rounds * (stages + start of a tile), both in units of a 128 x 256 stage: fitted to 300 layers (256 - 9000 rows, K 512 -
// 16384), 0.7 % off the best tile in the mean of 204 others and 14 % at the most (856 x 768 x 9088).  int8: from three quarters of the
// compute units' worth of 128 x 256 tiles; below that a compute unit has no second tile to overlap with and the smaller tiles of the other
// kernels win or lose by up to 1.2.  Those 204 layers (65 - 9000 rows, bf16 and fp32 output, static and per-token steps): 1.14 times as fast as
// the tile kernel in the mean with whole N, 1.23 with odd N, two slower by more than 2 % (856 x 768 x 9088 15.4 us, 14.3 there; 6018 x 1024 x
// 896 13.3, 12.8).  E4M3: the tile kernel has 256 x 256 tiles, with half the operand bytes per product; where
// they fill the rounds and K is long they are as quick (2818 x 4096 x 16384 183 us there, 190 here; 4608 x 3072 x 12288 167 and 149),
// so the fill of the rounds, weighted by the length of the K loop, is compared with the tile kernel's score (mfma_fp8_pick_score, 1 =
// full rounds of 256 x 256).  900 layers (65 - 9000 rows, K 512 - 16384, N 384 - 16384): the 148 taken are 1.17 times as fast in the mean, the
// slowest 0.98; of those not taken 121 would be faster by more than 2 %, small ones (765 x 512 x 3267 7.1 us, 9.2 there).
int pair_pick(const GemmArgs& a, const GemmTable& tb, OutMode mode, bool fp8) {
  if (a.M <= 64 || !pair_supported(a, tb, mode, 1, fp8)) return -1;
  static const float kStage[3] = {1.0f, 0.84f, 0.61f}, kStart[3] = {2.1f, 1.2f, 1.06f};
  static const float kStageFp8[3] = {1.0f, 0.76f, 0.62f}, kStartFp8[3] = {0.0f, 1.6f, 0.7f};
  const long cus = device_cus(), nk = a.K >> 7;
  auto tiles = [&](int bn) { return (long)((a.M + 127) / 128) * ((a.N + bn - 1) / bn); };
  if (4 * tiles(256) < 3 * cus) return -1;
  int best = -1;
  float best_cost = 0.0f, fill = 0.0f;
  for (int t = fp8 ? 1 : 0; t < 3; ++t) {
    const int bn = 256 - 64 * t;
    const long rounds = (tiles(bn) + cus - 1) / cus;
    const float cost = (float)rounds * ((float)nk * (fp8 ? kStageFp8 : kStage)[t] + (fp8 ? kStartFp8 : kStart)[t]);
    if (best < 0 || cost < best_cost) {
      best = t;
      best_cost = cost;
      fill = (float)((double)a.M * a.N / ((double)rounds * cus * 128 * bn)) * (t == 2 ? 0.95f : 1.0f);
    }
  }
  if (fp8 && fill * 0.92f * (1.0f + 2.0f / (float)nk) < mfma_fp8_pick_score(a, tb)) return -1;
  return best;
}

// Row tiles of a panel.  Each XCD walks an eighth of the tile list; where the list has about two, four or eight panels, all XCDs or every
// second one begin theirs at the same columns, and go on reading the same lines of W and writing the same columns of y at the same
// time, which costs most where y is most of the traffic.  E4M3, panels of eight / six: 8518 x 1664 x 14912 (67 row tiles) 275 / 208 us;
// fp32 output, K = 1408, N = 15936, 10 - 72 row tiles: eight 1.26 - 1.53 times the best width from 58 to 69 and 1.21 at 32, six 1.0 - 1.03
// there; K = 2048 or 3072 with bf16 output: at most 1.04.  Of 220 layers 38 change: 16 become faster by more than 3 %, one slower by 2 %.
// Up to 8 MB of W panels of six gain nothing (19 layers, 0.97 - 1.06 times the time; 8500 x 1536 x 4608 with its quantizer 76.9 / 77.5 us).
static int panel_rows(const GemmArgs& a) {
  bool same_columns = false;
  for (int panels = 2; panels <= 8; panels *= 2)
    same_columns = same_columns || (10 * a.tiles_m >= 72 * panels && 9 * a.tiles_m <= 80 * panels);
  const int rows = same_columns && (long long)a.N * a.K > (8 << 20) ? 6 : 8;
  return a.tiles_m < rows ? a.tiles_m : rows;
}

template <int BN>
static hipError_t launch_bn(GemmArgs a, float sp, bool bf, bool fp8, hipStream_t st) {
  a.tiles_m = (a.M + 127) / 128;
  a.tiles_n = (a.N + BN - 1) / BN;
  a.group_m = panel_rows(a);
  const long tiles = (long)a.tiles_m * a.tiles_n, cus = device_cus();
  const int grid = (int)(tiles < cus ? tiles : cus);
#define SQ_P(T, F, B) hipLaunchKernelGGL((seglinear_pair_kernel<BN, T, F, B>), dim3(grid), dim3(512), 0, st, a, sp)
  if (fp8) {
    if constexpr (BN < 256) { if (bf) SQ_P(false, true, true); else SQ_P(false, true, false); }
  } else if (a.tok_steps != nullptr) {
    if (bf) SQ_P(true, false, true); else SQ_P(true, false, false);
  } else {
    if (bf) SQ_P(false, false, true); else SQ_P(false, false, false);
  }
#undef SQ_P
  return hipGetLastError();
}

hipError_t launch_seglinear_pair(const GemmArgs& a, const GemmTable& tb, OutMode mode, int tile, bool fp8, hipStream_t st) {
  if (!pair_supported(a, tb, mode, tile, fp8)) return hipErrorInvalidConfiguration;
  const bool bf = mode == OUT_BF16;
  if (tile == 0) return launch_bn<256>(a, tb.s_pos[0], bf, fp8, st);
  if (tile == 1) return launch_bn<192>(a, tb.s_pos[0], bf, fp8, st);
  return launch_bn<128>(a, tb.s_pos[0], bf, fp8, st);
}

}  // namespace sq
