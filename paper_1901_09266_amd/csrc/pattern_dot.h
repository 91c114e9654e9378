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

template <int ST>
struct Load;
template <>
struct Load<DODE_F64> {
  __device__ static double get(const void* W, int64_t i, const float*, int64_t) {
    return static_cast<const double*>(W)[i];
  }
};
template <>
struct Load<DODE_F32> {
  __device__ static float get(const void* W, int64_t i, const float*, int64_t) {
    return static_cast<const float*>(W)[i];
  }
};
template <>
struct Load<DODE_BF16> {
  __device__ static float get(const void* W, int64_t i, const float*, int64_t) {
    return bf16_bits_to_f32(static_cast<const uint16_t*>(W)[i]);
  }
};
template <>
struct Load<DODE_FP8_E4M3> {
  __device__ static float get(const void* W, int64_t i, const float* scale, int64_t si) {
    return e4m3_bits_to_f32(static_cast<const uint8_t*>(W)[i]) * scale[si];
  }
};

// Two neighbouring values i, i+1 (i even) with one load.
template <int ST>
struct Load2;
template <>
struct Load2<DODE_F64> {
  __device__ static void get(const void* W, int64_t i, const float*, int64_t, int64_t, double& w0,
                             double& w1) {
    const double2 v = *reinterpret_cast<const double2*>(static_cast<const double*>(W) + i);
    w0 = v.x;
    w1 = v.y;
  }
};
template <>
struct Load2<DODE_F32> {
  __device__ static void get(const void* W, int64_t i, const float*, int64_t, int64_t, float& w0,
                             float& w1) {
    const float2 v = *reinterpret_cast<const float2*>(static_cast<const float*>(W) + i);
    w0 = v.x;
    w1 = v.y;
  }
};
template <>
struct Load2<DODE_BF16> {
  __device__ static void get(const void* W, int64_t i, const float*, int64_t, int64_t, float& w0,
                             float& w1) {
    const uint32_t b = *reinterpret_cast<const uint32_t*>(static_cast<const uint16_t*>(W) + i);
    w0 = bf16_bits_to_f32(static_cast<uint16_t>(b & 0xFFFFu));
    w1 = bf16_bits_to_f32(static_cast<uint16_t>(b >> 16));
  }
};
template <>
struct Load2<DODE_FP8_E4M3> {
  __device__ static void get(const void* W, int64_t i, const float* scale, int64_t si0, int64_t si1,
                             float& w0, float& w1) {
    const uint16_t b = *reinterpret_cast<const uint16_t*>(static_cast<const uint8_t*>(W) + i);
    w0 = e4m3_bits_to_f32(static_cast<uint8_t>(b & 0xFFu)) * scale[si0];
    w1 = e4m3_bits_to_f32(static_cast<uint8_t>(b >> 8)) * scale[si1];
  }
};

// Row (h, a) of rho_c applied to q_d:  sum_l sum_{p in row a} W[l][h-l][a,p] q[h-l][p].
// The row's entries are taken in CSR order from the link-sliced layout, where
// they come in pairs: one load brings two values (and one their two ODs), and
// the loads of four entries are issued together (the sums keep their order).
template <int ST, typename S>
__device__ __forceinline__ S row_dot(const DevPat& pt, const DevVals& v, int c, int h, int a,
                                     const S* q, int64_t q_t, int64_t q_b) {
  S acc = 0;
  const int32_t deg = pt.row_ptr[a + 1] - pt.row_ptr[a];
  const int32_t s0 = pt.sr_first[a];
  for (int l = 0; l < pt.K; ++l) {
    const int t = h - l;
    if (t < 0) break;
    if (t >= pt.T) continue;
    const int64_t base = c * v.cstride_r + ((int64_t)l * pt.T + t) * pt.sr_len;
    const int64_t sbase = (c * (int64_t)pt.K * pt.T + (int64_t)l * pt.T + t) * v.n_ptile;
    const S* qt = q + (int64_t)t * q_t;
    int32_t k = 0;
    for (; k + 4 <= deg; k += 4) {
      const int32_t slot = s0 + 64 * k;   // entries k, k+1; k+2, k+3 one pair further
      const int2 p01 = *reinterpret_cast<const int2*>(pt.sr_col + slot);
      const int2 p23 = *reinterpret_cast<const int2*>(pt.sr_col + slot + 128);
      S w0, w1, w2, w3;
      Load2<ST>::get(v.W, base + slot, v.scale, sbase + (p01.x >> 6), sbase + (p01.y >> 6), w0, w1);
      Load2<ST>::get(v.W, base + slot + 128, v.scale, sbase + (p23.x >> 6), sbase + (p23.y >> 6), w2,
                     w3);
      const S x0 = qt[col_at(p01.x, q_b)], x1 = qt[col_at(p01.y, q_b)];
      const S x2 = qt[col_at(p23.x, q_b)], x3 = qt[col_at(p23.y, q_b)];
      acc += w0 * x0;
      acc += w1 * x1;
      acc += w2 * x2;
      acc += w3 * x3;
    }
    if (k + 2 <= deg) {
      const int32_t slot = s0 + 64 * k;
      const int2 p01 = *reinterpret_cast<const int2*>(pt.sr_col + slot);
      S w0, w1;
      Load2<ST>::get(v.W, base + slot, v.scale, sbase + (p01.x >> 6), sbase + (p01.y >> 6), w0, w1);
      const S x0 = qt[col_at(p01.x, q_b)], x1 = qt[col_at(p01.y, q_b)];
      acc += w0 * x0;
      acc += w1 * x1;
      k += 2;
    }
    if (k < deg) {
      const int32_t slot = s0 + 64 * k;
      const int p = pt.sr_col[slot];
      acc += static_cast<S>(Load<ST>::get(v.W, base + slot, v.scale, sbase + (p >> 6))) *
             qt[col_at(p, q_b)];
    }
  }
  return acc;
}

// Column (t, p) of rho_c^T applied to residual rows: sum over lags l whose row
// block h = t+l is in the minibatch (slot_of_lag(l) >= 0) of sum_{a on p} W[l][t][a,p] r[slot][a].
// The column's entries are taken in CSC order from the OD-sliced layout, four
// steps' loads issued together.
template <int ST, typename S, typename F>
__device__ __forceinline__ S col_dot(const DevPat& pt, const DevVals& v, int c, int t, int p,
                                     F&& slot_of_lag, const S* Rd, int64_t r_s, int64_t r_b) {
  S acc = 0;
  const int32_t deg = pt.col_ptr[p + 1] - pt.col_ptr[p];
  const int32_t s0 = pt.sc_off[p >> 6] + (p & 63);
  for (int l = 0; l < pt.K; ++l) {
    const int h = t + l;
    if (h >= pt.H) break;
    const int s = slot_of_lag(l);
    if (s < 0) continue;
    const int64_t base = c * v.cstride_c + ((int64_t)l * pt.T + t) * pt.sc_len;
    const int64_t si = (c * (int64_t)pt.K * pt.T + (int64_t)l * pt.T + t) * v.n_ptile + (p >> 6);
    const S* r = Rd + (int64_t)s * r_s;
    int32_t k = 0;
    for (; k + 4 <= deg; k += 4) {
      S w[4], x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int32_t slot = s0 + 64 * (k + u);
        w[u] = static_cast<S>(Load<ST>::get(v.WT, base + slot, v.scale, si));
        x[u] = r[col_at(pt.sc_row[slot], r_b)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc += w[u] * x[u];
    }
    for (; k < deg; ++k) {
      const int32_t slot = s0 + 64 * k;
      acc += static_cast<S>(Load<ST>::get(v.WT, base + slot, v.scale, si)) * r[col_at(pt.sc_row[slot], r_b)];
    }
  }
  return acc;
}

// col_dot for the minibatch at positions first..first+bh-1 of a permutation
// with inverse pos_c (nullptr: every interval, slot h).
template <int ST, typename S>
__device__ __forceinline__ S col_dot_chunk(const DevPat& pt, const DevVals& v, int c, int t, int p,
                                           const int32_t* pos_c, int32_t first, int32_t bh,
                                           const S* Rd, int64_t r_s, int64_t r_b) {
  return col_dot<ST, S>(pt, v, c, t, p, [&](int l) {
    const int s = pos_c ? pos_c[t + l] - first : t + l;
    return s < bh ? s : -1;
  }, Rd, r_s, r_b);
}

}  // namespace
