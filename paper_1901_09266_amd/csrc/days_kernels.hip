// Matrix-core kernels of the pattern form for the days of one cluster: the
// products and adjoints of whole days (dode_apply, dode_loss, dode_grad,
// dode_metrics, dode_loss_bwd, the loss history of spgd_run) and the
// minibatches of FP32 and FP64 plans.  Products and sums are in the state
// type: v_mfma_f32_16x16x4_f32, or v_mfma_f64_16x16x4_f64 for FP64 handles.
//
// Tiles: 16 lines (links of the product, ODs of the adjoint) by the union of
// the columns that any of them has an entry in, four columns a group, made
// once per handle from the pattern (unions.hip).  The values are kept packed in
// operand order, runs of 16 columns, so a column group is one coalesced load;
// gathered from the sliced copies instead, the 64 values of a group lie in up to
// 64 cache lines (ODs: 950 against 553 us of the one-line-per-lane form below).
// Stored per entry, by link / by OD, with the padding of tiles and runs: corridor
// 400 x 1500 8% 1.3 / 1.5, 150 x 500 8% 2.0 / 2.4, 50 x 200 10% 2.8 / 4.1;
// independent incidence 150 x 500 8% 9.0 / 9.2, 3% 12.1 / 12.8.  A block owns one
// row block (interval h, departure interval t) for ND = 16 NT days: it stages the
// state rows its lags need in LDS, days fastest, and its waves take the tiles in
// turn.
//
// v_mfma_f32_16x16x4_f32 adds its four products to the accumulator one after
// the other, each with one rounding (fused multiply-add, increasing k), and a
// zero of the padding adds nothing.  Lag by lag and in increasing column order
// the sums are therefore the bits of the pattern walk (row_dot, col_dot), for
// any number of days.
//
// A tile's padding is zero; where a state value is not finite its product with
// the padding would reach lines the pattern does not connect, so entries that
// come out non-finite are formed again from the pattern alone (redo).
//
// One line per lane and one day per block (plain_kernels.hip) loads a value, an
// index and a state entry from cache per product: 400 days of 150 ODs, 500
// links, 288 intervals and 6 lags took 5.37 ms (product) and 3.41 ms (adjoint)
// in FP32; several days per lane from LDS 0.88 and 0.55 ms.
#include "dode_internal.h"
#include "pattern_dot.h"

namespace {

// waves of a block: the product's blocks come two to a CU, the adjoint's are
// held by the LDS of their longer rows
constexpr int kRowWaves = 8, kColWaves = 16;
constexpr int64_t kFillBlocks = 512;   // blocks that fill the chip
// 16-day tiles per block: with two, half the blocks and value loads, but the
// block's LDS doubles; 0.61 against 0.46 ms (product), 0.64 against 0.52 ms
// (adjoint) at 400 days of 150 ODs and 500 links
constexpr int kDayTiles = 1;
constexpr size_t kLdsBytes = 160 * 1024 - 4096;   // what a block may stage
constexpr size_t kStageBytes = 64 * 1024;         // what leaves room for a second block

template <typename S>
struct Vec;
template <>
struct Vec<float> {
  typedef float V4 __attribute__((ext_vector_type(4)));
  typedef float V4u __attribute__((ext_vector_type(4), aligned(4)));
  __device__ static V4 mma(float a, float b, V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct Vec<double> {
  typedef double V4 __attribute__((ext_vector_type(4)));
  typedef double V4u __attribute__((ext_vector_type(4), aligned(8)));
  __device__ static V4 mma(double a, double b, V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};

// Cluster, first day and day count of group g.
template <int ND>
__device__ __forceinline__ void day_group(const DayList& dl, int g, int& c, int& first, int& cnt) {
  if (dl.tab) {
    c = dl.tab[g];
    first = dl.tab[dl.n + g];
    cnt = dl.tab[2 * dl.n + g];
  } else {
    c = dl.cluster;
    first = g * ND;
    cnt = min(ND, dl.n_days - first);
  }
}

// Blocks in the order (row, group), groups fastest and a contiguous range per
// XCD: the groups of a cluster read the row's values from one L2.
__device__ __forceinline__ int xcd_item(int n) {
  const int per = (n + 7) / 8;
  return (blockIdx.x % 8) * per + blockIdx.x / 8;
}

// col_at in 32 bits: a staged row of all days fits them (lines <= 2496)
__device__ __forceinline__ uint32_t col32(int k, int64_t sb) {
  return (uint32_t)(k >> 2) * (uint32_t)sb + (k & 3);
}

// Stage one state row of the group's days, src[day d][column], as
// dst[column][day]: the columns 64 at a time (chunk), one per lane.  The day's
// row is a uniform address, the lane adds its column's 32-bit offset.
template <typename S, int ND>
__device__ __forceinline__ void stage_chunk(S* __restrict__ dst, const S* __restrict__ src,
                                            int64_t day_stride, int64_t sb, int n_cols, int cnt,
                                            int chunk) {
  typedef S V __attribute__((ext_vector_type(16 / sizeof(S))));
  constexpr int N = 16 / sizeof(S);
  const int p = chunk * 64 + (threadIdx.x & 63);
  if (p >= n_cols) return;
  const uint32_t o = col32(p, sb);
  S x[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    x[d] = d < cnt ? src[o] : S(0);
    src += day_stride;
  }
  V* q = reinterpret_cast<V*>(dst + p * ND);
#pragma unroll
  for (int i = 0; i < ND / N; ++i) {
    V v;
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = x[i * N + j];
    q[i] = v;
  }
}

// Four values of the consecutive lines l0..l0+3 at p, or of the lines line[0..3]
// of the same row (p is the row's column 0; sb the block stride of col_at).
template <typename S>
__device__ __forceinline__ typename Vec<S>::V4 get4(const S* __restrict__ p, const int* line,
                                                    bool run, int64_t sb) {
  if (run) {
    const auto v = *reinterpret_cast<const typename Vec<S>::V4u*>(p + col32(line[0], sb));
    return typename Vec<S>::V4{v[0], v[1], v[2], v[3]};
  }
  typename Vec<S>::V4 v;
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = line[k] >= 0 ? p[col32(line[k], sb)] : S(0);
  return v;
}

template <typename S>
__device__ __forceinline__ void put4(S* __restrict__ p, const typename Vec<S>::V4& v,
                                     const int* line, bool run, int64_t sb) {
  if (run) {
    *reinterpret_cast<typename Vec<S>::V4u*>(p + col32(line[0], sb)) =
        typename Vec<S>::V4u{v[0], v[1], v[2], v[3]};
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (line[k] >= 0) p[col32(line[k], sb)] = v[k];
}

template <typename V4>
__device__ __forceinline__ bool all_finite(const V4& v) {
  return __builtin_isfinite(v[0]) && __builtin_isfinite(v[1]) && __builtin_isfinite(v[2]) &&
         __builtin_isfinite(v[3]);
}

// The products of one tile with the staged rows of n_lags lags, lag by lag and
// in increasing column order:
// acc[u] += sum over lags i and columns k of value(i, k) * st[i][col k][16u + n].
// block(i) is the (uniform) block l*T + t of lag i, counted from the cluster's
// first; its packed values are vals + block * len.
// A step is one run of 16 columns of one lag: two loads (values, places), four
// LDS reads, four products, no branch.  kAhead steps are in flight, so a wave
// keeps a few KB of values on their way; with one test per column group each
// product waited for its own LDS read (2.7 times the matrix-core time).
template <int ST, typename S, int NT, typename B, typename F>
__device__ __forceinline__ void tile_product(const DevUnion& un, int tile, int n_lags, int n_cols,
                                             const S* st, const void* vals, int64_t len, B&& block,
                                             F&& scale, typename Vec<S>::V4* acc) {
  using E = typename Load<ST>::E;
  struct alignas(4 * sizeof(E)) E4 {
    E v[4];
  };
  constexpr int ND = 16 * NT, kAhead = 4;
  struct Step {
    int4 at;
    E4 w;
    int i;   // lag
  };
  const uint32_t lane = threadIdx.x & 63;
  const int n = lane & 15, kg = lane >> 4;
  const int r_begin = un.off[tile], r_end = un.off[tile + 1];
  const int n_steps = (r_end - r_begin) * n_lags;
  if (n_steps <= 0) return;
  int i = 0, r = r_begin;   // the next step to load
  const E4* base = static_cast<const E4*>(vals) + block(0) * (len / 4);
  auto load = [&](Step& q) {   // past the last step: its places again
    q.at = reinterpret_cast<const int4*>(un.col)[(uint32_t)(4 * r + kg)];
    q.w = base[(uint32_t)(64 * r) + lane];
    q.i = i;
    if (++r == r_end) {
      if (i + 1 < n_lags) {
        r = r_begin;
        base = static_cast<const E4*>(vals) + block(++i) * (len / 4);
      } else {
        r = r_end - 1;
      }
    }
  };
  auto use = [&](const Step& q, bool on) {
    const S* row = st + (int64_t)q.i * n_cols * ND + n;
    const int at[4] = {q.at.x, q.at.y, q.at.z, q.at.w};
    S x[4][NT];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int u = 0; u < NT; ++u) x[j][u] = row[at[j] * ND + 16 * u];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      S a = Load<ST>::raw(q.w.v[j]);
      if constexpr (ST == DODE_FP8_E4M3) a *= scale(block(q.i), at[j]);
      a = on ? a : S(0);
#pragma unroll
      for (int u = 0; u < NT; ++u) acc[u] = Vec<S>::mma(a, x[j][u], acc[u]);
    }
  };
  Step q[kAhead];
#pragma unroll
  for (int k = 0; k < kAhead; ++k) load(q[k]);
  for (int s = 0; s < n_steps; s += kAhead) {
#pragma unroll
    for (int k = 0; k < kAhead; k += 2) {   // two steps at a time, the second may be past the end
      if (s + k >= n_steps) break;
      use(q[k], true);
      use(q[k + 1], s + k + 1 < n_steps);
      load(q[k]);
      load(q[k + 1]);
    }
  }
}

// Product rows of the groups' days: out = rho_c Q (- X if X) for the row
// blocks of cs (cs.perm == nullptr: every interval), and, with PART, the
// FP64 sums of squares of each (day, interval).
template <int ST, typename S, int NT, bool PART>
__global__ void __launch_bounds__(64 * kRowWaves)
k_rows_days(DevPat pt, DevVals v, DevUnion un, DayList dl, ChunkSched cs, int n_rows, Layout ly,
            int64_t o_d, int64_t o_r, int64_t o_b, int kl, const S* __restrict__ Q,
            const S* __restrict__ X, S* __restrict__ out, double* __restrict__ part) {
  using V4 = typename Vec<S>::V4;
  constexpr int ND = 16 * NT;
  extern __shared__ __align__(16) unsigned char stage_mem[];
  S* st = reinterpret_cast<S*>(stage_mem);
  __shared__ double sh[PART ? kRowWaves * ND : 1];
  const int item = xcd_item(n_rows * dl.n);
  if (item >= n_rows * dl.n) return;
  const int s = item / dl.n;
  int c, first, cnt;
  day_group<ND>(dl, item - s * dl.n, c, first, cnt);
  int h = s;
  if (cs.perm) {
    if (cs.j0 + s >= pt.H) return;
    cs = resolve_epoch(cs);
    h = cs.perm[c * pt.H + cs.j0 + s];
  }
  const int tid = threadIdx.x, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, kg = lane >> 4;
  // lags with t = h - l inside [0, T)
  const int l_lo = h - pt.T + 1 > 0 ? h - pt.T + 1 : 0;
  const int l_hi = h < pt.K - 1 ? h : pt.K - 1;
  const int64_t cblk = (int64_t)c * pt.K * pt.T;
  double ss[NT];
  const S* xp[NT];
  S* op[NT];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int64_t day = first + 16 * u + n;
    ss[u] = 0.0;
    xp[u] = X + day * ly.x_d + (int64_t)h * ly.x_h;
    op[u] = out + day * o_d + (int64_t)s * o_r;
  }
  bool staged = false;
  // this block's part of the tiles
  const int per = (un.n_tiles + gridDim.y - 1) / gridDim.y;
  const int t_begin = blockIdx.y * per, t_end = min(un.n_tiles, t_begin + per);
  for (int t0 = t_begin; t0 < t_end; t0 += nw) {
    const int tile = t0 + wave;
    V4 acc[NT], x[NT];
    int line[4] = {-1, -1, -1, -1};
    bool run = false;
    if (tile < t_end) {
#pragma unroll
      for (int k = 0; k < 4; ++k) line[k] = un.line[16 * tile + 4 * kg + k];
      run = un.run[4 * tile + kg];
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) {   // the observed rows come while the product runs
      acc[u] = x[u] = V4{};
      if (X && tile < t_end && 16 * u + n < cnt) x[u] = get4(xp[u], line, run, ly.x_b);
    }
    for (int lc = l_lo; lc <= l_hi; lc += kl) {
      const int le = min(l_hi + 1, lc + kl);
      if (!staged) {
        if (lc != l_lo || t0 > t_begin) __syncthreads();   // the last stage has been read
        const int nc = (pt.P + 63) / 64;
        for (int i = wave; i < (le - lc) * nc; i += nw) {
          const int li = i / nc;
          stage_chunk<S, ND>(st + (int64_t)li * pt.P * ND,
                             Q + first * ly.q_d + (int64_t)(h - lc - li) * ly.q_t, ly.q_d, ly.q_b,
                             pt.P, cnt, i - li * nc);
        }
        __syncthreads();
        staged = lc == l_lo && le > l_hi;   // every lag fits: staged once
      }
      if (tile < t_end)
        tile_product<ST, S, NT>(
            un, tile, le - lc, pt.P, st, v.PR, v.pr_len,
            [&](int i) { return cblk + (int64_t)(lc + i) * pt.T + h - lc - i; },
            [&](int64_t b, int p) { return v.scale[b * v.n_ptile + (p >> 6)]; }, acc);
    }
    if (tile >= t_end) continue;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (16 * u + n >= cnt) continue;
      V4 val = acc[u];
      if (!all_finite(val))
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (!__builtin_isfinite(val[k]) && line[k] >= 0)
            val[k] = row_dot<ST, S>(pt, v, c, h, line[k],
                                    Q + (int64_t)(first + 16 * u + n) * ly.q_d, ly.q_t, ly.q_b);
      if (X) val -= x[u];
      if (out) put4(op[u], val, line, run, o_b);
      if constexpr (PART) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (line[k] >= 0) ss[u] += static_cast<double>(val[k]) * static_cast<double>(val[k]);
      }
    }
  }
  if constexpr (PART) {
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      ss[u] += __shfl_xor(ss[u], 16, 64);
      ss[u] += __shfl_xor(ss[u], 32, 64);
      if (kg == 0) sh[wave * ND + 16 * u + n] = ss[u];
    }
    __syncthreads();
    if (tid < cnt) {
      double r = 0.0;
      for (int w = 0; w < nw; ++w) r += sh[w * ND + tid];
      part[(int64_t)(first + tid) * pt.H + h] = r;
    }
  }
}

// Position of the i-th set bit of m.
__device__ __forceinline__ int nth_bit(uint64_t m, int i) {
  for (; i > 0; --i) m &= m - 1;
  return __builtin_ctzll(m);
}

// Adjoint rows of the groups' days.  STEP: the departure intervals a minibatch
// reaches (cs), with the Adagrad or fixed step and the projection on Q and A;
// otherwise Q[t] = f * rho_c^T R for every t.
template <int ST, typename S, int NT, bool STEP>
__global__ void __launch_bounds__(64 * kColWaves)
k_cols_days(DevPat pt, DevVals v, DevUnion un, DayList dl, ChunkSched cs, int n_rows, Layout ly,
            int kl, const S* __restrict__ R, S* __restrict__ Q, S* __restrict__ A, StepArgs sa,
            double f) {
  using V4 = typename Vec<S>::V4;
  constexpr int ND = 16 * NT;
  extern __shared__ __align__(16) unsigned char stage_mem[];
  S* st = reinterpret_cast<S*>(stage_mem);
  const int item = xcd_item(n_rows * dl.n);
  if (item >= n_rows * dl.n) return;
  const int row = item / dl.n;
  int c, first, cnt;
  day_group<ND>(dl, item - row * dl.n, c, first, cnt);
  int t = row;
  uint64_t lags = 0;   // lags whose rows are reached
  const int32_t* dsc = nullptr;
  if constexpr (STEP) {
    cs = resolve_epoch(cs);
    dsc = cs.touched + ((int64_t)c * cs.max_touched + row) * desc_width(pt.K);
    t = dsc[kDescT];
    if (t < 0) return;
    lags = (uint64_t)(uint32_t)dsc[kDescMask] | (uint64_t)(uint32_t)dsc[kDescMask + 1] << 32;
  } else {
    const int m = min(pt.K, pt.H - t);
    lags = m >= 64 ? ~0ull : m <= 0 ? 0 : (1ull << m) - 1;
  }
  const int tid = threadIdx.x, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, kg = lane >> 4;
  const int n_lags = __popcll(lags);
  const int64_t cblk = (int64_t)c * pt.K * pt.T;
  bool staged = false;
  const int per = (un.n_tiles + gridDim.y - 1) / gridDim.y;
  const int t_begin = blockIdx.y * per, t_end = min(un.n_tiles, t_begin + per);
  for (int t0 = t_begin; t0 < t_end; t0 += nw) {
    const int tile = t0 + wave;
    V4 acc[NT];
    int line[4] = {-1, -1, -1, -1};
    bool run = false;
    if (tile < t_end) {
#pragma unroll
      for (int k = 0; k < 4; ++k) line[k] = un.line[16 * tile + 4 * kg + k];
      run = un.run[4 * tile + kg];
    }
    const int64_t qd = (int64_t)(first + n) * ly.q_d + (int64_t)t * ly.q_t;
#pragma unroll
    for (int u = 0; u < NT; ++u) acc[u] = V4{};
    uint64_t m = lags;   // lags still to do
    for (int lc = 0; lc < n_lags; lc += kl) {
      const int nl = min(kl, n_lags - lc);
      if (!staged) {
        if (lc > 0 || t0 > t_begin) __syncthreads();
        const int nc = (pt.L + 63) / 64;
        for (int i = wave; i < nl * nc; i += nw) {
          const int li = i / nc;
          const int l = nth_bit(m, li);
          const int64_t slot = STEP ? dsc[kDescSlot + l] : t + l;
          stage_chunk<S, ND>(st + (int64_t)li * pt.L * ND, R + first * ly.r_d + slot * ly.r_s,
                             ly.r_d, ly.r_b, pt.L, cnt, i - li * nc);
        }
        __syncthreads();
        staged = lc == 0 && nl == n_lags;
      }
      if (tile < t_end)
        tile_product<ST, S, NT>(
            un, tile, nl, pt.L, st, v.PC, v.pc_len,
            [&](int i) { return cblk + (int64_t)nth_bit(m, i) * pt.T + t; },
            [&](int64_t b, int) {   // FP8: the tile row's OD has the scale
              return v.scale[b * v.n_ptile + (max(0, un.line[16 * tile + n]) >> 6)];
            },
            acc);
      for (int i = 0; i < nl; ++i) m &= m - 1;
    }
    if (tile >= t_end) continue;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (16 * u + n >= cnt) continue;
      const int64_t day = first + 16 * u + n;
      V4 g = acc[u];
      if (!all_finite(g))
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (!__builtin_isfinite(g[k]) && line[k] >= 0)
            g[k] = col_dot<ST, S>(pt, v, c, t, line[k], [&](int l) {
              return !STEP ? t + l : (lags >> l & 1) ? (int)dsc[kDescSlot + l] : -1;
            }, R + day * ly.r_d, ly.r_s, ly.r_b);
      S* qp = Q + qd + 16 * u * ly.q_d;
      if constexpr (STEP) {
        V4 q = get4(qp, line, run, ly.q_b);
        if (sa.optimizer == 0) {
          V4 a = get4(A + qd + 16 * u * ly.q_d, line, run, ly.q_b);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            a[k] += g[k] * g[k];
            q[k] -= static_cast<S>(sa.eta) * g[k] / (sqrt(a[k]) + static_cast<S>(sa.eps));
          }
          put4(A + qd + 16 * u * ly.q_d, a, line, run, ly.q_b);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) q[k] -= static_cast<S>(sa.eta) * g[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = q[k] > S(0) ? q[k] : S(0);
        put4(qp, q, line, run, ly.q_b);
      } else {
        if (f != 1.0)
#pragma unroll
          for (int k = 0; k < 4; ++k) g[k] = static_cast<S>(static_cast<double>(g[k]) * f);
        put4(qp, g, line, run, ly.q_b);
      }
    }
  }
}

int lag_chunk(int K, int cols, size_t row_bytes) {
  return std::max(1, std::min<int>(K, (int)(kStageBytes / (cols * row_bytes))));
}

// Grid of a launch and its block size.  The blocks of a short minibatch leave
// CUs idle while each walks its tiles in several rounds of its waves: they are
// then split into parts that stage the rows again (with 45 blocks of 17 tiles,
// 13.0 against 8.3 us per launch).
dim3 grid_of(int n_rows, const DayList& dl, const DevUnion& un, int waves, bool split,
             unsigned* threads) {
  const int64_t blocks = ((int64_t)n_rows * dl.n + 7) / 8 * 8;
  int64_t parts = 1;
  if (split)
    parts = std::max<int64_t>(1, std::min<int64_t>((un.n_tiles + waves - 1) / waves, kFillBlocks / blocks));
  const int per = (int)((un.n_tiles + parts - 1) / parts);
  *threads = 64u * std::min(per, waves);
  return dim3((unsigned)blocks, (unsigned)parts);
}

template <int ST, typename S, int NT>
hipError_t rows(const dode_dar* dar, const DayList& dl, const ChunkSched& cs, int n_rows,
                const Layout& ly, int64_t o_d, int64_t o_r, int64_t o_b, const void* Q,
                const void* X, void* out, double* part, hipStream_t s) {
  const size_t rb = 16 * NT * sizeof(S);
  const int kl = lag_chunk(dar->dims.K, dar->dims.P, rb);
  const size_t lds = (size_t)kl * dar->dims.P * rb;
  const DevUnion& un = dar->u_rows;
  unsigned threads = 0;
  // the row sums of `part` need all of a row's tiles in one block
  const dim3 grid = grid_of(n_rows, dl, un, kRowWaves, part == nullptr, &threads);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(threads), lds, s,
                       dar->pat(), dar->vals(), un, dl, cs, n_rows, ly, o_d, o_r, o_b, kl,
                       static_cast<const S*>(Q), static_cast<const S*>(X), static_cast<S*>(out),
                       part);
  };
  if (part)
    go(k_rows_days<ST, S, NT, true>);
  else
    go(k_rows_days<ST, S, NT, false>);
  return hipGetLastError();
}

template <int ST, typename S, int NT, bool STEP>
hipError_t cols(const dode_dar* dar, const DayList& dl, const ChunkSched& cs, int n_rows,
                const Layout& ly, const void* R, void* Q, void* A, const StepArgs& sa, double f,
                hipStream_t s) {
  const size_t rb = 16 * NT * sizeof(S);
  // a minibatch reaches an interval through one or two of its lags
  const int kl = lag_chunk(STEP ? std::min(2, dar->dims.K) : dar->dims.K, dar->dims.L, rb);
  const size_t lds = (size_t)kl * dar->dims.L * rb;
  const DevUnion& un = dar->u_cols;
  unsigned threads = 0;
  const dim3 grid = grid_of(n_rows, dl, un, kColWaves, true, &threads);
  hipLaunchKernelGGL((k_cols_days<ST, S, NT, STEP>), grid, dim3(threads), lds, s, dar->pat(), dar->vals(), un, dl, cs,
                     n_rows, ly, kl, static_cast<const S*>(R), static_cast<S*>(Q), static_cast<S*>(A), sa, f);
  return hipGetLastError();
}

// f<ST, S> of the handle's storage
template <typename F>
hipError_t by_storage(const dode_dar* dar, F&& f) {
  switch (dar->storage) {
    case DODE_F64: return f(std::integral_constant<int, DODE_F64>{}, 0.0);
    case DODE_F32: return f(std::integral_constant<int, DODE_F32>{}, 0.f);
    case DODE_BF16: return f(std::integral_constant<int, DODE_BF16>{}, 0.f);
    default: return f(std::integral_constant<int, DODE_FP8_E4M3>{}, 0.f);
  }
}

}  // namespace

// ---- which form a call takes ----------------------------------------------
// The one-day kernels cost what the days' entries cost, the 16-day kernels what
// the union tiles do, padding included, for groups that may be nearly empty, and
// small launches of either are a chain of round trips.  No single count decides
// it: by products alone (2^22 a pass; 2^20 an epoch and 32 days in groups half
// full) a loss over one day of 400 ODs, 1500 links, 96 intervals with 5%
// independent incidence took 219 us against 94 one day per block (FP32), an epoch
// of 32 days of 150 ODs, 500 links, 3% incidence in minibatches of 4 of 144
// intervals 1444 against 558 us (FP64).  So both are estimated, in us, and the
// smaller is taken.  The models were fitted to launches in 3 to 288 intervals of 1
// to 200 days, 26 x 300 to 400 x 1500 networks with corridor and independent
// incidence (standard deviation 0.2 to 0.35 of the time); the faster
// form against the one taken, geometric means: 0.99 over 1704 epochs in FP32 and
// FP64, 0.99 over 772 losses, 0.98 over 772 gradients in all four types.
namespace {

// Stored types in the order of dode_dtype.
struct FormCost {
  double row_step, row_stage, col_step, col_stage, col_base;   // 16 days, per block
  double pass_row, pass_col, pass_chain;                       // one day, whole passes
  double step_row, step_col;                                   // one day, minibatches
};
constexpr FormCost kCost[] = {
    {0.19, 0.44, 0.22, 0.46, 9.0, 0.74, 1.05, 0.5, 0.35, 0.80},
    {0.19, 0.20, 0.30, 0.12, 6.0, 0.56, 0.73, 0.5, 0.30, 0.49},
    {0.18, 0.20, 0.22, 0.35, 5.0, 0.51, 0.72, 0.5, 0.30, 0.49},
    {0.73, 0.15, 1.00, 0.50, 4.0, 0.62, 0.77, 0.7, 0.30, 0.49},
};
constexpr double kFullWaves = 3200;     // waves that keep their latency to themselves
constexpr double kBytesPerUs = 5.0e6;   // packed values from memory
// Whole passes take less than the model, which minibatches are most of: a gradient
// of 400 ODs, 1500 links, 96 intervals, 1 day in FP32 53 us against 78 one day per
// block, where the plain comparison takes the latter.
constexpr double kPass = 0.8;

// One launch of a 16-day kernel: `lags` lags of each of n_rows rows of `groups` day
// groups in `clusters` clusters.  A block's longest wave takes `step` per column
// run and lag and the block `stage` per 64 columns and lag it stages, again for
// every round of its tiles where the lags do not fit at once; past kFullWaves
// they queue. The packed values come from memory once per cluster.
double group_launch(const dode_dar* dar, const DevUnion& un, int64_t len, int waves, bool split,
                    double n_rows, int64_t groups, int64_t clusters, double lags, int cols, int kl,
                    double step, double stage, double base) {
  const double blocks = n_rows * groups;
  const int rounds = (un.n_tiles + waves - 1) / waves;
  const double parts =
      split ? std::max(1.0, std::min<double>(rounds, std::floor(kFillBlocks / std::max(1.0, blocks)))) : 1.0;
  const int w = std::min(un.n_tiles, waves);
  const double again = lags <= kl ? 1.0 : std::ceil(rounds / parts);
  const double block = step * (len / 256.0) * lags / w / parts + stage * lags * again * cols / 64.0 + base;
  const double bytes = (double)clusters * n_rows * lags * len * dar->value_size;
  return block * std::max(1.0, blocks * parts * w / kFullWaves) + bytes / kBytesPerUs;
}

double group_rows(const dode_dar* dar, double n_rows, int64_t groups, int64_t clusters, bool split) {
  const FormCost& c = kCost[dar->storage];
  const size_t rb = 16 * kDayTiles * (is_f64(dar) ? 8 : 4);
  return group_launch(dar, dar->u_rows, dar->pr_len, kRowWaves, split, n_rows, groups, clusters,
                      dar->dims.K, dar->dims.P, lag_chunk(dar->dims.K, dar->dims.P, rb), c.row_step,
                      c.row_stage, 5.0);
}

double group_cols(const dode_dar* dar, double n_rows, int64_t groups, int64_t clusters, double lags,
                  bool step) {
  const FormCost& c = kCost[dar->storage];
  const size_t rb = 16 * kDayTiles * (is_f64(dar) ? 8 : 4);
  const int kl = lag_chunk(step ? std::min(2, dar->dims.K) : dar->dims.K, dar->dims.L, rb);
  return group_launch(dar, dar->u_cols, dar->pc_len, kColWaves, true, n_rows, groups, clusters, lags,
                      dar->dims.L, kl, c.col_step, c.col_stage, c.col_base);
}

// A link's (OD's) walk over its lags, eight entries a step, and the work of
// n_rows rows of every day, in million slots.
double row_chain(const dode_dar* dar) {
  return (dar->dims.L + 255) / 256 * dar->dims.K * ((dar->max_row + 3) / 4);
}
double mega_slots(const dode_dar* dar, int64_t slots, double n_rows, int64_t days) {
  return 1e-6 * slots * dar->dims.K * n_rows * days;
}

}  // namespace

bool day_launch_fits(int32_t n_rows, int64_t groups, int32_t n_tiles, bool rows) {
  return (n_rows * groups + 7) / 8 * 8 * 64 * std::min(n_tiles, rows ? kRowWaves : kColWaves) <=
         kGridThreads;
}

bool day_rows_fit(const dode_dar* dar) {
  const size_t lines = std::max(dar->dims.P, dar->dims.L);
  return lines * 16 * kDayTiles * (is_f64(dar) ? 8 : 4) <= kLdsBytes;
}

bool day_groups_fit(const dode_dar* dar, int64_t groups) {
  return day_rows_fit(dar) && day_launch_fits(dar->dims.H, groups, dar->u_rows.n_tiles, true) &&
         day_launch_fits(dar->dims.T, groups, dar->u_cols.n_tiles, false);
}

int32_t days_per_group() { return 16 * kDayTiles; }

bool group_rows_pay(const dode_dar* dar, int64_t groups, int64_t clusters, int64_t days, bool sums) {
  const FormCost& c = kCost[dar->storage];
  return kPass * group_rows(dar, dar->dims.H, groups, clusters, !sums) <
         c.pass_row * mega_slots(dar, dar->row_slots, dar->dims.H, days) + 0.14 * row_chain(dar);
}

bool group_cols_pay(const dode_dar* dar, int64_t groups, int64_t clusters, int64_t days) {
  const FormCost& c = kCost[dar->storage];
  const double chain = (dar->dims.P + 63) / 64 * dar->dims.K * ((dar->max_col + 7) / 8);
  return kPass * group_cols(dar, dar->dims.T, groups, clusters, dar->dims.K, false) <
         c.pass_col * mega_slots(dar, dar->col_slots, dar->dims.T, days) + c.pass_chain * chain;
}

bool group_step_pays(const dode_dar* dar, int32_t bh, int32_t touched, int64_t groups,
                     int64_t clusters, int64_t days) {
  const FormCost& c = kCost[dar->storage];
  const double lags = (double)dar->dims.K * bh / std::max(1, touched);   // per reached interval
  return group_rows(dar, bh, groups, clusters, true) + group_cols(dar, touched, groups, clusters, lags, true) <
         c.step_row * mega_slots(dar, dar->row_slots, bh, days) + 0.07 * row_chain(dar) +
             c.step_col * mega_slots(dar, dar->col_slots, bh, days) +
             0.4 * lags * ((dar->max_col + 7) / 8) + 5.3;
}

bool groups_ever_pay(const dode_dar* dar) {
  const int64_t groups = 256, days = groups * days_per_group();
  return group_rows_pay(dar, groups, 1, days, true) || group_rows_pay(dar, groups, 1, days, false) ||
         group_cols_pay(dar, groups, 1, days) ||
         group_step_pays(dar, dar->dims.H, dar->dims.T, groups, 1, days);
}

hipError_t days_rows(const dode_dar* dar, const DayList& dl, const ChunkSched* cs, int32_t n_rows,
                     const Layout& ly, const void* Q, const void* X, void* out, double* part,
                     hipStream_t s) {
  const ChunkSched c0 = cs ? *cs : ChunkSched{};
  // a minibatch writes residual rows (R, row = slot), whole days X rows (row = h)
  const int64_t o_d = cs ? ly.r_d : ly.x_d, o_r = cs ? ly.r_s : ly.x_h, o_b = cs ? ly.r_b : ly.x_b;
  return by_storage(dar, [&](auto st, auto state) {
    return rows<decltype(st)::value, decltype(state), kDayTiles>(
        dar, dl, c0, n_rows, ly, o_d, o_r, o_b, Q, X, out, part, s);
  });
}

hipError_t days_cols(const dode_dar* dar, const DayList& dl, const Layout& ly, const void* R,
                     void* G, double f, hipStream_t s) {
  return by_storage(dar, [&](auto st, auto state) {
    return cols<decltype(st)::value, decltype(state), kDayTiles, false>(
        dar, dl, ChunkSched{}, dar->dims.T, ly, R, G, nullptr, StepArgs{}, f, s);
  });
}

hipError_t days_cols_step(const dode_dar* dar, const DayList& dl, const ChunkSched& cs,
                          const Layout& ly, const void* R, void* Q, void* A, const StepArgs& sa,
                          hipStream_t s) {
  return by_storage(dar, [&](auto st, auto state) {
    return cols<decltype(st)::value, decltype(state), kDayTiles, true>(
        dar, dl, cs, cs.max_touched, ly, R, Q, A, sa, 1.0, s);
  });
}
