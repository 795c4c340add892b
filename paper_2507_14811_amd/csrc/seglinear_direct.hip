// SegLinear + DualScale GEMM for small layers (embedding and conditioning projections: some dozens to hundreds of token rows, a
// short reduction): a wave per 32 x 32 block of outputs, operands straight into registers.
//
// Such a layer is a chain of latencies, not work: 64 x 256 x 384 in two K-segments took the K-splitting kernel 8.1 us, a trip to
// memory, a barrier per stage and an exchange through LDS per K-segment, on six tiles.  Here nothing is shared and nothing
// waits but a wave for its own operands: all of the layer's constants and the first four 128-byte stages are requested at
// once, the ring of four stages runs on across the K-segments (both operands keep the same order of k, and a segment boundary
// only scales the sums), and 24 waves on as many compute units finish after one trip.
// What bounds it beyond that is the loads: a lane reads 16 bytes of one of 32 rows, so that an instruction touches 32 lines, and
// every wave fetches its operands itself: few waves or short reductions only (direct_pick).
// 64 x 256 x 384: 6.9 -> 4.3 us in a stream of launches.
#include "seglinear_mfma_kernel.hpp"

namespace sq {

constexpr int kDirectSegments = 2, kDirectRing = 4;
struct DirectTable {
  int S, seg_end, dual[kDirectSegments];     // seg_end: stages of 128 columns in the first of two K-segments
  float s_pos[kDirectSegments], s_neg[kDirectSegments];
};

template <bool DUAL>
__global__ __launch_bounds__(64) void seglinear_direct_kernel(const GemmArgs a, const DirectTable tb, const int mode) {
  const int lane = threadIdx.x, row = lane & 31, kg = lane >> 5;
  const int n0 = blockIdx.x * 32, m = blockIdx.y * 32 + row;
  const int mr = m < a.M ? m : a.M - 1, nr = n0 + row < a.N ? n0 + row : a.N - 1;   // ragged edges: the last row again, masked at the store
  const int8_t* px = a.xq + (size_t)mr * a.K + 16 * kg;
  const int8_t* pw = a.wq + (size_t)nr * a.K + 16 * kg;
  const int nst = a.K >> 7, nc = n0 + 4 * kg;                       // this lane's columns: nc + 8 g + i (g, i < 4)
  const bool inside = n0 + 32 <= a.N && a.N % 4 == 0 &&             // whole, aligned row pieces
                      ((reinterpret_cast<uintptr_t>(a.y) | reinterpret_cast<uintptr_t>(a.wscale) | reinterpret_cast<uintptr_t>(a.bias)) % 16 == 0);
  struct Cols { float v[16]; };
  auto columns = [&](const float* p) __attribute__((always_inline)) {
    Cols c;
    if (inside) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4f t = *reinterpret_cast<const v4f*>(p + nc + 8 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) c.v[4 * g + i] = t[i];
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int n = nc + 8 * (v >> 2) + (v & 3);
        c.v[v] = p[n < a.N ? n : a.N - 1];
      }
    }
    return c;
  };
  v4i x[kDirectRing][4], w[kDirectRing][4];
  auto load = [&](const int j, const int stage) __attribute__((always_inline)) {   // beyond the last stage: that one again
    const int at = (stage < nst ? stage : nst - 1) * 128;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      x[j][h] = *reinterpret_cast<const v4i*>(px + at + 32 * h);
      w[j][h] = *reinterpret_cast<const v4i*>(pw + at + 32 * h);
    }
  };
  // the constants first: loads return in order
  Cols cw[kDirectSegments] = {columns(a.wscale), columns(a.wscale + (tb.S > 1 ? a.N : 0))};
  const Cols bias = columns(a.bias != nullptr ? a.bias : a.wscale);
  float sp[kDirectSegments], sn[kDirectSegments];
#pragma unroll
  for (int s = 0; s < kDirectSegments; ++s) {
    const int ks = s < tb.S ? s : 0;
    const bool dl = DUAL && tb.dual[ks] != 0;
    sp[s] = tb.s_pos[ks];
    sn[s] = dl ? tb.s_neg[ks] : 0.0f;
    if (a.tok_steps) {                                              // dynamic per-token steps of this lane's row
      sp[s] = a.tok_steps[(size_t)mr * tb.S + ks];
      sn[s] = dl ? a.tok_steps[((size_t)a.M + mr) * tb.S + ks] : 0.0f;
    }
  }
#pragma unroll
  for (int j = 0; j < kDirectRing; ++j) load(j, j);

  v16i accp = (v16i)(0), accn = (v16i)(0);
  float sum[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) sum[v] = a.bias != nullptr ? bias.v[v] : 0.0f;
  const int boundary = tb.S > 1 ? tb.seg_end : -1;
  bool dl = DUAL && tb.dual[0] != 0;
  auto flush = [&](const Cols& c, const float s_p, const float s_n) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int p = DUAL ? accp[v] - accn[v] : accp[v];             // X^_+ W^ = X^ W^ - X^_- W^, exactly (integers)
      float t = s_p * (float)p;
      if (DUAL) t = __builtin_fmaf(s_n, (float)accn[v], t);
      sum[v] = __builtin_fmaf(c.v[v], t, sum[v]);                   // two or three roundings per K-segment, the bias's among them
      accp[v] = 0;
      accn[v] = 0;
    }
  };
  for (int t = 0; t < nst; t += kDirectRing) {
#pragma unroll
    for (int j = 0; j < kDirectRing; ++j) {
      if (t + j < nst) {
        if (t + j == boundary) {                                    // a new K-segment: the sums of the first one are complete
          flush(cw[0], sp[0], sn[0]);
          dl = DUAL && tb.dual[1] != 0;
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) accp = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[j][h], x[j][h], accp, 0, 0, 0);
        if (DUAL && dl) {
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            v4i xn;
#pragma unroll
            for (int d = 0; d < 4; ++d) xn[d] = negative_codes(x[j][h][d]);
            accn = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[j][h], xn, accn, 0, 0, 0);
          }
        }
      }
      load(j, t + j + kDirectRing);
    }
  }
  if (tb.S > 1) flush(cw[1], sp[1], sn[1]);
  else flush(cw[0], sp[0], sn[0]);
  if (m >= a.M) return;
  const size_t o = (size_t)m * a.N + nc;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const float* t = sum + 4 * g;
    if (mode == OUT_BF16) {
      uint16_t* y = reinterpret_cast<uint16_t*>(a.y) + o + 8 * g;
      if (inside) {
        *reinterpret_cast<v2i*>(y) = (v2i){(int)f32x2_to_bf16x2(t[0], t[1]), (int)f32x2_to_bf16x2(t[2], t[3])};
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (nc + 8 * g + i < a.N) y[i] = f32_to_bf16(t[i]);
      }
    } else {
      float* y = reinterpret_cast<float*>(a.y) + o + 8 * g;
      if (inside) {
        *reinterpret_cast<v4f*>(y) = (v4f){t[0], t[1], t[2], t[3]};
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (nc + 8 * g + i < a.N) y[i] = t[i];
      }
    }
  }
}

bool direct_supported(const GemmArgs& a, const GemmTable& tb, OutMode mode) {
  if (tb.S > kDirectSegments || tb.has_seg_scale || mode == OUT_DEBUG_ACC) return false;
  for (int s = 0; s <= tb.S; ++s)
    if (tb.kseg_off[s] % 128 != 0) return false;
  return (a.M + 31) / 32 <= 65535 && (reinterpret_cast<uintptr_t>(a.xq) | reinterpret_cast<uintptr_t>(a.wq)) % 16 == 0;
}

// Where it is the faster one, by the waves (blocks of 32 x 32) and the columns.  Measured on 700 layers of 33 - 1024 rows, 128 - 4096
// outputs and 128 - 16384 columns against what ran before, mostly the K-splitting kernel.  Two K-segments, for each of which that
// kernel starts and exchanges anew: a wave per compute unit at most, two polarity paths 6.9 -> 4.4 us (64 x 256 x 384), 17.3 -> 12.4
// (70 x 4096 x 512), even at 8192 columns (23.3 / 21.1) and behind beyond (25.5 / 25.0 at 10240); one path 11.7 -> 9.7 at 4096; two
// waves per compute unit 14.0 -> 11.6 (128 x 2048 x 4096), 17.8 / 18.8 at 4096 columns; at four they share the loads' path (256 x 256
// x 4096: 7.7 / 9.1).  One K-segment: two paths 5.1 -> 4.1 at 512 columns, 8.9 -> 7.8 at 2048, 11.7 / 12.3 at 4096; one path 3.9 / 3.9
// at 256, 4.3 -> 3.9 at 384, 6.4 -> 5.6 at 1536, 7.2 / 7.1 at 2048.
// Up to 32 rows come here where the slab of the weight-stream kernel is too small for them (17 - 32 rows from 2560 columns, 1 - 16
// from 5120).  With per-token steps the K-splitting kernel would run: 1.06 - 2.2 times as fast here (125 layers).  With static steps it
// is the skinny kernel, whose four waves split K: of 58 layers of 16 rows and fewer most are slower here (0.82 - 1.1, median 0.94), so
// they stay there.  17 - 32 rows, 400 layers: beyond 4096 outputs 1.6 - 1.9 times as fast (24 x 6272 x 8192 31.6 -> 17.9 us), without
// a split segment 1.0 - 1.16; below, where at least half of the columns run two paths, 0.99 - 1.19 up to 4096 columns or 1024 outputs
// and 0.93 - 1.14 (median 1.0) beyond both; 0.84 - 1.2 (median 1.01) where less than half do.
bool direct_pick(const GemmArgs& a, const GemmTable& tb, OutMode mode) {
  if (!direct_supported(a, tb, mode)) return false;
  const long long waves = (long long)((a.M + 31) / 32) * ((a.N + 31) / 32);
  const int cus = device_cus();
  bool dual = false;
  int split = 0;                                                    // columns of two paths
  for (int s = 0; s < tb.S; ++s) {
    if (!tb.dual[s]) continue;
    dual = true;
    split += tb.kseg_off[s + 1] - tb.kseg_off[s];
  }
  if (a.M <= 32 && a.tok_steps == nullptr &&
      (a.M <= 16 || (a.N <= 4096 && (2 * split < a.K || (a.K > 4096 && a.N > 1024)))))
    return false;
  if (tb.S == 2) return a.K <= 2048 ? waves <= 2 * cus : waves <= cus && a.K <= (dual ? 8192 : 4096);
  return waves <= cus && (dual ? a.K <= 2048 : a.K >= 384 && a.K <= 1536);
}

hipError_t launch_seglinear_direct(const GemmArgs& a, const GemmTable& tb, OutMode mode, hipStream_t st) {
  if (!direct_supported(a, tb, mode)) return hipErrorInvalidConfiguration;
  DirectTable dt{};
  dt.S = tb.S;
  dt.seg_end = tb.kseg_off[1] >> 7;
  bool dual = false;
  for (int s = 0; s < tb.S; ++s) {
    dt.dual[s] = tb.dual[s];
    dt.s_pos[s] = tb.s_pos[s];
    dt.s_neg[s] = tb.s_neg[s];
    dual = dual || tb.dual[s] != 0;
  }
  const dim3 grid((a.N + 31) / 32, (a.M + 31) / 32);
  if (dual) hipLaunchKernelGGL(seglinear_direct_kernel<true>, grid, dim3(64), 0, st, a, dt, (int)mode);
  else hipLaunchKernelGGL(seglinear_direct_kernel<false>, grid, dim3(64), 0, st, a, dt, (int)mode);
  return hipGetLastError();
}

}  // namespace sq
