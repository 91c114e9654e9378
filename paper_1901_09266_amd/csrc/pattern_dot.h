// The pattern form of the assignment blocks: loads of stored values widened to
// the state type, and the walks of one output entry of rho_c q or rho_c^T r
// (entries in CSR / CSC order).
#pragma once

#include "dode_internal.h"

namespace {

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// OCP E4M3FN: 1 sign, 4 exponent bits (bias 7), 3 mantissa bits; exponent
// field 0 is subnormal (m * 2^-9); the all-ones code is NaN (never stored).
__device__ __forceinline__ float e4m3_bits_to_f32(uint8_t b) {
  const uint32_t e = (b >> 3) & 0xF, m = b & 7;
  float v = e == 0 ? static_cast<float>(m) * 0x1p-9f : __uint_as_float(((e + 120u) << 23) | (m << 20));
  return (b & 0x80) ? -v : v;
}

// Stored values widened to the state type: one, or a neighbouring pair.
// `scale` holds the FP8 scales of the value's block, one per 64 ODs; raw leaves
// the scale to the caller.
template <int ST>
struct Load;
template <>
struct Load<DODE_F64> {
  using E = double;
  using Pair = double2;
  __device__ static double raw(double w) { return w; }
  __device__ static double widen(double w, const float*, int) { return w; }
  __device__ static void widen(double2 w, const float*, int2, double& w0, double& w1) {
    w0 = w.x;
    w1 = w.y;
  }
};
template <>
struct Load<DODE_F32> {
  using E = float;
  using Pair = float2;
  __device__ static float raw(float w) { return w; }
  __device__ static float widen(float w, const float*, int) { return w; }
  __device__ static void widen(float2 w, const float*, int2, float& w0, float& w1) {
    w0 = w.x;
    w1 = w.y;
  }
};
template <>
struct Load<DODE_BF16> {
  using E = uint16_t;
  using Pair = uint32_t;
  __device__ static float raw(uint16_t w) { return bf16_bits_to_f32(w); }
  __device__ static float widen(uint16_t w, const float*, int) { return raw(w); }
  __device__ static void widen(uint32_t w, const float*, int2, float& w0, float& w1) {
    w0 = bf16_bits_to_f32(static_cast<uint16_t>(w & 0xFFFFu));
    w1 = bf16_bits_to_f32(static_cast<uint16_t>(w >> 16));
  }
};
template <>
struct Load<DODE_FP8_E4M3> {
  using E = uint8_t;
  using Pair = uint16_t;
  __device__ static float raw(uint8_t w) { return e4m3_bits_to_f32(w); }
  __device__ static float widen(uint8_t w, const float* scale, int tile) {
    return raw(w) * scale[tile];
  }
  __device__ static void widen(uint16_t w, const float* scale, int2 p, float& w0, float& w1) {
    w0 = e4m3_bits_to_f32(static_cast<uint8_t>(w & 0xFFu)) * scale[p.x >> 6];
    w1 = e4m3_bits_to_f32(static_cast<uint8_t>(w >> 8)) * scale[p.y >> 6];
  }
};

__device__ __forceinline__ float fma_s(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_s(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}

// Row a's products of lags [l_begin, l_end), NE entries (even) of every lag from
// entry k0 on.  The entries' columns are read once, and the values of LU lags
// are in flight together: a walk whose loads wait for each other spends its time
// on their latency.  `stage` runs once the first loads are issued (it may fill
// the LDS that q points to).  Past the row's last entry the last pair is read
// again and its product dropped.
template <int ST, typename S, int NE, int LU, typename F>
__device__ __forceinline__ S row_part(const DevPat& pt, const DevVals& v, int c, int h, int32_t deg,
                                      int32_t s0, int32_t k0, int l_begin, int l_end, const S* q,
                                      int64_t q_t, int64_t q_b, S acc, F&& stage) {
  using E = typename Load<ST>::E;
  int2 p[NE / 2];
  uint32_t slot[NE / 2];
#pragma unroll
  for (int j = 0; j < NE / 2; ++j) {
    slot[j] = s0 + 64 * max(0, min(k0 + 2 * j, (deg - 1) & ~1));
    p[j] = deg > 0 ? *reinterpret_cast<const int2*>(pt.sr_col + slot[j]) : make_int2(0, 0);
  }
  typename Load<ST>::Pair w[LU][NE / 2];
  auto fetch = [&](int l0) {
#pragma unroll
    for (int i = 0; i < LU; ++i) {
      const int l = l0 + i, t = h - l;
      if (l >= l_end) break;
      const E* W = static_cast<const E*>(v.W) + c * v.cstride_r + ((int64_t)l * pt.T + t) * pt.sr_len;
#pragma unroll
      for (int j = 0; j < NE / 2; ++j)
        if (deg > 0) w[i][j] = *reinterpret_cast<const typename Load<ST>::Pair*>(W + slot[j]);
    }
  };
  fetch(l_begin);
  stage();
  for (int l0 = l_begin; l0 < l_end; l0 += LU) {
#pragma unroll
    for (int i = 0; i < LU; ++i) {
      if (l0 + i >= l_end) break;
      const int t = h - l0 - i;
      const float* scale = v.scale + (c * (int64_t)pt.K * pt.T + (int64_t)(l0 + i) * pt.T + t) * v.n_ptile;
      const S* qt = q + (int64_t)t * q_t;
#pragma unroll
      for (int j = 0; j < NE / 2; ++j) {
        S w0, w1;
        Load<ST>::widen(w[i][j], scale, p[j], w0, w1);
        const S s = fma_s(w0, qt[col_at(p[j].x, q_b)], acc);
        acc = k0 + 2 * j < deg ? s : acc;
        const S u = fma_s(w1, qt[col_at(p[j].y, q_b)], acc);
        acc = k0 + 2 * j + 1 < deg ? u : acc;
      }
    }
    if (l0 + LU < l_end) fetch(l0 + LU);
  }
  return acc;
}

// Row (h, a) of rho_c applied to q_d:  sum_l sum_{p in row a} W[l][h-l][a,p] q[h-l][p],
// lags ascending, a lag's entries in CSR order, from the link-sliced layout
// (entries come in pairs).  ME is the longest row the form takes: up to 8
// entries three lags' loads go out together, up to 16 two lags', beyond that
// (ME = 0) eight entries of one lag (ME = -4: four, for kernels whose other work
// needs the registers).  any: false for a wave none of whose rows has entries.
template <int ST, typename S, int ME, typename F>
__device__ __forceinline__ S row_dot(const DevPat& pt, const DevVals& v, int c, int h, int32_t deg,
                                     int32_t s0, bool any, const S* q, int64_t q_t, int64_t q_b,
                                     F&& stage) {
  const int l_begin = max(0, h - pt.T + 1);   // t = h - l in [0, T)
  const int l_end = any ? min(pt.K, h + 1) : l_begin;
  S acc = 0;
  if constexpr (ME > 0) {
    return row_part<ST, S, ME, ME == 8 ? 3 : 2>(pt, v, c, h, deg, s0, 0, l_begin, l_end, q, q_t, q_b,
                                                acc, stage);
  } else {
    constexpr int NE = ME < 0 ? -ME : 8;
    stage();
    for (int l = l_begin; l < l_end; ++l)
      for (int32_t k = 0; k < deg; k += NE)
        acc = row_part<ST, S, NE, 1>(pt, v, c, h, deg, s0, k, l, l + 1, q, q_t, q_b, acc, [] {});
    return acc;
  }
}

template <int ST, typename S>
__device__ __forceinline__ S row_dot(const DevPat& pt, const DevVals& v, int c, int h, int a,
                                     const S* q, int64_t q_t, int64_t q_b) {
  return row_dot<ST, S, -4>(pt, v, c, h, pt.row_ptr[a + 1] - pt.row_ptr[a], pt.sr_first[a], true, q,
                           q_t, q_b, [] {});
}

// Column (t, p) of rho_c^T over the lags of `mask` (those whose rows are given),
// lags ascending, a lag's entries in CSC order, from the OD-sliced layout; row(n, l)
// is the residual row of the n-th set lag l.  `width` is the longest column of the
// wave's slice.  Entries go in steps of 8, three steps' loads in flight;
// `stage` runs once the first ones are issued.  Every lane reads `width` entries,
// its column's and then the slice's padding, so a load is a run of memory (with
// each lane's own last entry again instead, columns of unequal length cost 1.5
// times as much); the products past the column's end are dropped.
template <int ST, typename S, typename G, typename F>
__device__ __forceinline__ S col_walk(const DevPat& pt, const DevVals& v, int c, int t, int slice,
                                      int32_t deg, int32_t s0, int32_t width, uint64_t mask,
                                      int64_t r_b, G&& row, F&& stage) {
  using E = typename Load<ST>::E;
  constexpr int NE = 8, kSteps = 3;
  E w[kSteps][NE];
  int32_t a[kSteps][NE];
  uint64_t m = mask;   // of the next fetch
  int32_t kf = 0;
  auto fetch = [&](int b) {
    if (!m) return;
    const int l = __builtin_ctzll(m);
    const E* WT = static_cast<const E*>(v.WT) + c * v.cstride_c + ((int64_t)l * pt.T + t) * pt.sc_len;
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const uint32_t slot = s0 + 64 * min(kf + u, width - 1);
      w[b][u] = WT[slot];
      a[b][u] = pt.sc_row[slot];
    }
    kf += NE;
    if (kf >= width) {
      kf = 0;
      m &= m - 1;
    }
  };
  if (width == 0) m = 0;
#pragma unroll
  for (int b = 0; b < kSteps; ++b) fetch(b);
  stage();
  S acc = 0;
  uint64_t mu = width == 0 ? 0 : mask;   // of the next product
  int32_t k = 0;
  int n = 0;
  while (mu) {
#pragma unroll
    for (int b = 0; b < kSteps; ++b) {
      if (!mu) break;
      const int l = __builtin_ctzll(mu);
      const S* r = row(n, l);
      const float* scale = v.scale + (c * (int64_t)pt.K * pt.T + (int64_t)l * pt.T + t) * v.n_ptile;
#pragma unroll
      for (int u = 0; u < NE; ++u) {
        const S s = fma_s(Load<ST>::widen(w[b][u], scale, slice), r[col_at(a[b][u], r_b)], acc);
        acc = k + u < deg ? s : acc;
      }
      k += NE;
      if (k >= width) {
        k = 0;
        ++n;
        mu &= mu - 1;
      }
      fetch(b);
    }
  }
  return acc;
}

// Column (t, p) of rho_c^T applied to residual rows: sum over lags l whose row
// block h = t+l is in the minibatch (slot_of_lag(l) >= 0) of sum_{a on p} W[l][t][a,p] r[slot][a],
// in the order of col_walk.
template <int ST, typename S, typename F>
__device__ __forceinline__ S col_dot(const DevPat& pt, const DevVals& v, int c, int t, int p,
                                     F&& slot_of_lag, const S* Rd, int64_t r_s, int64_t r_b) {
  using E = typename Load<ST>::E;
  S acc = 0;
  const int32_t deg = pt.col_ptr[p + 1] - pt.col_ptr[p];
  const int32_t s0 = pt.sc_off[p >> 6] + (p & 63);
  for (int l = 0; l < pt.K; ++l) {
    const int h = t + l;
    if (h >= pt.H) break;
    const int s = slot_of_lag(l);
    if (s < 0) continue;
    const E* WT = static_cast<const E*>(v.WT) + c * v.cstride_c + ((int64_t)l * pt.T + t) * pt.sc_len;
    const float* scale = v.scale + (c * (int64_t)pt.K * pt.T + (int64_t)l * pt.T + t) * v.n_ptile;
    const S* r = Rd + (int64_t)s * r_s;
    for (int32_t k = 0; k < deg; k += 8) {
      E w[8];
      int32_t a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t slot = s0 + 64 * min(k + u, deg - 1);
        w[u] = WT[slot];
        a[u] = pt.sc_row[slot];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const S x = fma_s(Load<ST>::widen(w[u], scale, p >> 6), r[col_at(a[u], r_b)], acc);
        acc = k + u < deg ? x : acc;
      }
    }
  }
  return acc;
}

}  // namespace
