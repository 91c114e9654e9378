// Sparse (pattern-compact) kernels of libdode: the general path for every
// storage type.  Each thread owns one output entry and walks the pattern, so
// results are deterministic (fixed summation order, no atomics).
//
// Algorithm 1 (section "Non-negative least square on GPU") per minibatch:
//   chunk_resid   : r = rho_o q - x_o on the minibatch rows (eq. "finalobj")
//   chunk_adj_step: g = rho_o^T r, then Adagrad / fixed step and max(q, 0),
//                   fused, for every departure interval the minibatch reaches.
#include "dode_internal.h"
#include "pattern_dot.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int kRowsBlock = 256;
constexpr int kColsWaves = 4;
constexpr int kAdjBlock = 64;
constexpr int kRedBlock = 256;
constexpr size_t kStageBytes = 32768;   // rows of the other operand staged in LDS by a block

__device__ __forceinline__ int day_cl(const int32_t* day_cluster, int32_t cluster, int d) {
  return day_cluster ? day_cluster[d] : cluster;
}

// Fixed-order block sum of one double per thread (blockDim.x == kRedBlock).
__device__ double block_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int w = kRedBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  return sh[0];
}

// ------------------------------------------------------------- kernels --
// One link per thread, the lanes of a slice in the order of their slots (sr_lane),
// so a wave's loads of values are runs of memory: with the links in their own
// order every load took 16 instead of 4 cycles of the address unit, half of the
// kernel's time.  With STAGE the block copies the K demand rows its links read,
// Q_d[h-l] for l < K, into LDS (row l at l*P; rows outside the day are zeros
// that no lane reads) while the first values are on their way.  What is left is
// latency: table, permutation, then operands, then a round trip per two or three
// lags.  60 days of 50 ODs, 200 links, 6 lags, bf16, 40 intervals: 35.2 -> 21.2 us
// (29 MB of values).
template <int ST, typename S, bool STAGE, int ME>
__global__ void __launch_bounds__(kRowsBlock)
k_chunk_resid(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, ChunkSched cs,
              Layout ly, const S* __restrict__ Q, const S* __restrict__ X, S* __restrict__ R) {
  extern __shared__ unsigned char q_stage[];
  const int ln = blockIdx.x * kRowsBlock + threadIdx.x;
  const int s = blockIdx.y, d = blockIdx.z;
  cs = resolve_epoch(cs);
  const int c = day_cl(day_cluster, cluster, d);
  if (cs.j0 + s >= pt.H) return;   // the whole block
  const int h = cs.perm[c * pt.H + cs.j0 + s];
  const int4 lane = ln < (pt.L + 63) / 64 * 64 ? pt.sr_lane[ln] : make_int4(-1, 0, 0, 0);
  const int a = lane.x;
  const bool in = a >= 0;
  const int32_t deg = lane.y, s0 = lane.z;
  // a slice's links come by degree: a first lane without entries is a wave
  // without (the waves past the last slice are: half of a block with 83 links)
  const bool any = __builtin_amdgcn_readfirstlane(deg) > 0;
  const S x = in ? X[d * ly.x_d + h * ly.x_h + col_at(a, ly.x_b)] : S(0);
  S xhat;
  if constexpr (STAGE) {
    S* qs = reinterpret_cast<S*>(q_stage);
    const S* qd = Q + d * ly.q_d;
    const unsigned inv = 0xffffffffu / (unsigned)pt.P + 1;   // i / P while i * P < 2^32 (P > 1)
    // row t = h - l of the staged copy sits at (h - t) * P: base h*P, stride -P
    xhat = row_dot<ST, S, ME>(pt, v, c, h, deg, s0, any, qs + (int64_t)h * pt.P, -(int64_t)pt.P, 4, [&] {
      for (int i = threadIdx.x; i < pt.K * pt.P; i += kRowsBlock) {
        const int l = pt.P > 1 ? (int)__umulhi((unsigned)i, inv) : i, p = i - l * pt.P, t = h - l;
        qs[i] = (t >= 0 && t < pt.T) ? qd[(int64_t)t * ly.q_t + col_at(p, ly.q_b)] : S(0);
      }
      __syncthreads();
    });
  } else {
    xhat = row_dot<ST, S, ME>(pt, v, c, h, deg, s0, any, Q + d * ly.q_d, ly.q_t, ly.q_b, [] {});
  }
  if (in) R[d * ly.r_d + s * ly.r_s + col_at(a, ly.r_b)] = xhat - x;
}

// One column per thread; a wave takes the 64 columns of one slice in one
// reached interval and day, a block kColsWaves such tasks.  The wave copies the
// residual rows that reach the interval (the set bits of the descriptor's lag
// mask, in order) into its part of the LDS, so the walk's gathers are LDS reads
// and its only loads are the pattern's; an interval that more than `rows` of the
// minibatch's rows reach takes them from memory.  Descriptor, then rows and
// values together, then LDS: a walk that looked up each lag's position, then
// its links, then their residuals took a round trip for each (31.2 -> 26.4 us
// for 60 days of 50 ODs, 200 links, 40 of 288 intervals, bf16; residuals from
// memory in one-wave blocks 27.0).
template <int ST, typename S>
__global__ void __launch_bounds__(64 * kColsWaves)
k_chunk_adj_step(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, ChunkSched cs,
                 Layout ly, int rows, const S* __restrict__ R, S* __restrict__ Q,
                 S* __restrict__ A, StepArgs st) {
  extern __shared__ unsigned char r_stage[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int slices = (pt.P + 63) / 64, task = blockIdx.x * kColsWaves + wave;
  const int i = task / slices, p = 64 * (task - i * slices) + lane, d = blockIdx.y;
  if (i >= cs.max_touched) return;
  cs = resolve_epoch(cs);
  const int c = day_cl(day_cluster, cluster, d);
  const int32_t* dsc = cs.touched + ((int64_t)c * cs.max_touched + i) * desc_width(pt.K);
  const int slot_l = lane < pt.K ? dsc[kDescSlot + lane] : -1;
  const int slice = task - i * slices;
  const bool in = p < pt.P, adagrad = st.optimizer == 0;
  const int column = min(lane, pt.P - 1 - 64 * slice);   // lanes past the last OD read its values
  const int32_t deg = in ? pt.col_ptr[p + 1] - pt.col_ptr[p] : 0;
  const int32_t off = pt.sc_off[slice];
  const int32_t width = ((slice + 1 < slices ? pt.sc_off[slice + 1] : (int32_t)pt.sc_len) - off) / 64;
  const int t = dsc[kDescT];
  if (t < 0) return;
  const uint64_t mask = (uint64_t)(uint32_t)dsc[kDescMask] |
                        (uint64_t)(uint32_t)dsc[kDescMask + 1] << 32;
  const S* Rd = R + d * ly.r_d;
  const int64_t idx = d * ly.q_d + t * ly.q_t + col_at(p, ly.q_b);
  S q = in ? Q[idx] : S(0), acc = in && adagrad ? A[idx] : S(0), g;
  if (__builtin_popcountll(mask) <= rows) {
    S* rs = reinterpret_cast<S*>(r_stage) + (int64_t)wave * rows * pt.L;
    g = col_walk<ST, S>(pt, v, c, t, slice, deg, off + column, width, mask, 4,
                        [&](int n, int) { return rs + n * pt.L; }, [&] {
      S* to = rs;
      for (uint64_t m = mask; m;) {
        // two rows, four values of each per lane in flight
        const S* r0 = Rd + (int64_t)__builtin_amdgcn_readlane(slot_l, __builtin_ctzll(m)) * ly.r_s;
        m &= m - 1;
        const bool two = m != 0;
        const S* r1 = two ? Rd + (int64_t)__builtin_amdgcn_readlane(slot_l, __builtin_ctzll(m)) * ly.r_s : r0;
        m &= m - 1;
        for (int a = lane; a < pt.L; a += 256) {
          S x[4], y[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (a - lane + 64 * u >= pt.L) break;
            const int64_t k = col_at(min(a + 64 * u, pt.L - 1), ly.r_b);
            x[u] = r0[k];
            if (two) y[u] = r1[k];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (a + 64 * u >= pt.L) break;
            to[a + 64 * u] = x[u];
            if (two) to[pt.L + a + 64 * u] = y[u];
          }
        }
        to += 2 * pt.L;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    });
  } else {
    g = col_walk<ST, S>(pt, v, c, t, slice, deg, off + column, width, mask, ly.r_b, [&](int, int l) {
      return Rd + (int64_t)__builtin_amdgcn_readlane(slot_l, l) * ly.r_s;
    }, [] {});
  }
  if (!in) return;
  if (adagrad) {
    acc += g * g;
    A[idx] = acc;
    q -= static_cast<S>(st.eta) * g / (sqrt(acc) + static_cast<S>(st.eps));
  } else {
    q -= static_cast<S>(st.eta) * g;
  }
  Q[idx] = q > S(0) ? q : S(0);
}

template <int ST, typename S>
__global__ void __launch_bounds__(kRedBlock)
k_apply_rows(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, Layout ly,
             const S* __restrict__ Q, const S* __restrict__ X, S* __restrict__ out,
             double* __restrict__ part) {
  __shared__ double sh[kRedBlock];
  const int h = blockIdx.x, d = blockIdx.y;
  const int c = day_cl(day_cluster, cluster, d);
  const S* q = Q + d * ly.q_d;
  double ss = 0.0;
  for (int a = threadIdx.x; a < pt.L; a += kRedBlock) {
    S val = row_dot<ST, S>(pt, v, c, h, a, q, ly.q_t, ly.q_b);
    const int64_t o = d * ly.x_d + h * ly.x_h + col_at(a, ly.x_b);
    if (X) val -= X[o];
    if (out) out[o] = val;
    ss += static_cast<double>(val) * static_cast<double>(val);
  }
  if (part) {
    const double tot = block_sum(ss, sh);
    if (threadIdx.x == 0) part[(int64_t)d * pt.H + h] = tot;
  }
}

// One wave per departure interval and day.  (col_walk over every lag with a wave
// per slice was slower, 23.0 against 20.9 us for 18 days of 26 ODs, 483 links, 24
// intervals, 6 lags: its registers cost waves, and the residuals come from memory.)
template <int ST, typename S>
__global__ void __launch_bounds__(kAdjBlock)
k_adjoint_rows(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, Layout ly,
               const S* __restrict__ R, S* __restrict__ G) {
  const int t = blockIdx.x, d = blockIdx.y;
  const int c = day_cl(day_cluster, cluster, d);
  const S* Rd = R + d * ly.r_d;
  for (int p = threadIdx.x; p < pt.P; p += kAdjBlock)
    G[d * ly.q_d + t * ly.q_t + col_at(p, ly.q_b)] =
        col_dot<ST, S>(pt, v, c, t, p, [&](int l) { return t + l; }, Rd, ly.r_s, ly.r_b);
}

// One wave per day: lane i takes partials i, i+64, ..., then a butterfly (fixed
// order).  One thread per day left a serial chain of 288 loads: 22 us for any
// number of days.
__global__ void __launch_bounds__(kRedBlock)
k_sum_partials(const double* __restrict__ part, int32_t n_per, int32_t n_days,
               double* __restrict__ out, const int32_t* __restrict__ order) {
  const int d = blockIdx.x * (kRedBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (d >= n_days) return;
  double s = 0.0;
  for (int i = lane; i < n_per; i += 64) s += part[(int64_t)d * n_per + i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) out[order ? order[d] : d] = s;
}

__global__ void __launch_bounds__(kRedBlock)
k_max_partials(const double* __restrict__ part, int32_t n_per, int32_t n_days,
               double* __restrict__ out) {
  const int d = blockIdx.x * (kRedBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (d >= n_days) return;
  double m = 0.0;
  for (int i = lane; i < n_per; i += 64) m = fmax(m, part[(int64_t)d * n_per + i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if (lane == 0) out[d] = m;
}

// One wave per row of a day (four per block), eight values per lane in flight,
// then a butterfly: a block per row spent its time in the barriers of its tree
// (400 days of 288 rows of 150: 85 -> 32 us; of 500: 107 -> 65 us per pass).
constexpr int kRowAhead = 8;
template <typename S>
__global__ void __launch_bounds__(kRedBlock)
k_kkt_partials(const S* __restrict__ Q, const S* __restrict__ G, int32_t T, int32_t P,
               double* __restrict__ part) {
  const int t = blockIdx.x * (kRedBlock / 64) + (threadIdx.x >> 6), d = blockIdx.y;
  const int lane = threadIdx.x & 63;
  if (t >= T) return;
  const int64_t row = ((int64_t)d * T + t) * P;
  double m = 0.0;
  for (int p0 = lane; p0 < P; p0 += 64 * kRowAhead) {
    S q[kRowAhead], g[kRowAhead];
#pragma unroll
    for (int u = 0; u < kRowAhead; ++u) {
      const int p = p0 + 64 * u;
      q[u] = p < P ? Q[row + p] : S(0);
      g[u] = p < P ? G[row + p] : S(0);
    }
#pragma unroll
    for (int u = 0; u < kRowAhead; ++u) {
      const double a = q[u], b = g[u];
      m = fmax(m, fabs(a < b ? a : b));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if (lane == 0) part[(int64_t)d * T + t] = m;
}

// First pass (sum_x == nullptr): per (d, h) sum of x.  Second pass: sum of (x - mean)^2.
template <typename S>
__global__ void __launch_bounds__(kRedBlock)
k_x_moment(const S* __restrict__ X, int32_t H, int32_t L, const double* __restrict__ sum_x,
           double* __restrict__ part) {
  const int h = blockIdx.x * (kRedBlock / 64) + (threadIdx.x >> 6), d = blockIdx.y;
  const int lane = threadIdx.x & 63;
  if (h >= H) return;
  const double mean = sum_x ? sum_x[d] / (static_cast<double>(H) * L) : 0.0;
  const S* row = X + ((int64_t)d * H + h) * L;
  double s = 0.0;
  for (int a0 = lane; a0 < L; a0 += 64 * kRowAhead) {
    S v[kRowAhead];
#pragma unroll
    for (int u = 0; u < kRowAhead; ++u) v[u] = a0 + 64 * u < L ? row[a0 + 64 * u] : S(0);
#pragma unroll
    for (int u = 0; u < kRowAhead; ++u) {
      if (a0 + 64 * u >= L) continue;
      const double x = v[u];
      s += sum_x ? (x - mean) * (x - mean) : x;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) part[(int64_t)d * H + h] = s;
}

__global__ void k_r2(const double* loss, const double* sst, int32_t n, double* r2) {
  const int d = blockIdx.x * blockDim.x + threadIdx.x;
  if (d < n) r2[d] = 1.0 - loss[d] / sst[d];
}

// Bound by memory: 631 MB of FP32 in 164 us (187 with one value per load and
// thread, 190 with four vectors a grid's width apart in flight).
template <typename S>
__global__ void __launch_bounds__(256)
k_check_finite(const S* __restrict__ X, int64_t n, int32_t* flag) {
  constexpr int W = 16 / sizeof(S), U = 4;   // 16-byte loads, four in flight
  typedef S V __attribute__((ext_vector_type(W), aligned(sizeof(S))));
  const V* xv = reinterpret_cast<const V*>(X);
  const int64_t nv = n / W, first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  for (int64_t b = blockIdx.x; b * U * 256 < nv; b += gridDim.x) {   // U * 4 KB per block
    const int64_t i = b * U * 256 + threadIdx.x;
    if (i + (U - 1) * 256 < nv) {
      V x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = xv[i + u * 256];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < W; ++k) bad |= !isfinite(x[u][k]);
    } else {
      for (int64_t e = i; e < nv; e += 256)
#pragma unroll
        for (int k = 0; k < W; ++k) bad |= !isfinite(xv[e][k]);
    }
  }
  if (first < n - nv * W) bad |= !isfinite(X[nv * W + first]);
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

template <typename S>
__global__ void k_clamp(S* __restrict__ Q, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    Q[i] = Q[i] > S(0) ? Q[i] : S(0);
}

template <template <int, typename> class F, typename... Args>
hipError_t dispatch(const dode_dar* dar, Args&&... args) {
  switch (dar->storage) {
    case DODE_F64: return F<DODE_F64, double>::run(args...);
    case DODE_F32: return F<DODE_F32, float>::run(args...);
    case DODE_BF16: return F<DODE_BF16, float>::run(args...);
    case DODE_FP8_E4M3: return F<DODE_FP8_E4M3, float>::run(args...);
  }
  return hipErrorInvalidValue;
}

template <int ST, typename S>
struct RunResid {
  static hipError_t run(const dode_dar* dar, const int32_t* dc, int32_t cl, const ChunkSched& cs,
                        const Layout& ly, const void* Q, const void* X, void* R, int32_t n,
                        hipStream_t s) {
    dim3 grid((dar->dims.L + kRowsBlock - 1) / kRowsBlock, cs.bh, n);
    const size_t stage = (size_t)dar->dims.K * dar->dims.P * sizeof(S);
    auto go = [&](auto kern, size_t lds) {
      hipLaunchKernelGGL(kern, grid, dim3(kRowsBlock), lds, s, dar->pat(), dar->vals(), dc, cl, cs,
                         ly, static_cast<const S*>(Q), static_cast<const S*>(X), static_cast<S*>(R));
    };
    // The forms of 8 and 16 entries hide latency at 60 to 150 registers, 3 to 8
    // blocks a CU.  A launch of more blocks than that is better off with four
    // entries of a lag at a time where their entries are mostly padding (links of
    // 2.5 ODs, at most 9: 96 intervals of 60 days in FP64 37 against 51 us an
    // epoch, of 4 days 20 either way; links of 5 ODs, at most 14: 40 intervals of
    // 365 days in FP32 1484 against 1349), and for the 16 in FP8, whose codes cost
    // most to widen (40 intervals of 60 days 461 against 509, 10 870 against 750).
    const int64_t me = dar->max_row <= 8 ? 8 : 16;
    const bool fills = (int64_t)grid.x * grid.y * grid.z >= 1024;
    const bool padded = me * dar->dims.L > 5 * dar->nnz || (me == 16 && ST == DODE_FP8_E4M3);
    if (stage > kStageBytes)
      go(k_chunk_resid<ST, S, false, 0>, 0);
    else if (dar->max_row > 16)
      go(k_chunk_resid<ST, S, true, 0>, stage);
    else if (fills && padded)
      go(k_chunk_resid<ST, S, true, -4>, stage);
    else if (me == 8)
      go(k_chunk_resid<ST, S, true, 8>, stage);
    else
      go(k_chunk_resid<ST, S, true, 16>, stage);
    return hipGetLastError();
  }
};

template <int ST, typename S>
struct RunAdjStep {
  static hipError_t run(const dode_dar* dar, const int32_t* dc, int32_t cl, const ChunkSched& cs,
                        const Layout& ly, const void* R, void* Q, void* A, int32_t n,
                        const StepArgs& st, hipStream_t s) {
    const int64_t tasks = (int64_t)(dar->dims.P + 63) / 64 * cs.max_touched;
    dim3 grid((unsigned)((tasks + kColsWaves - 1) / kColsWaves), n);
    const int64_t row = (int64_t)dar->dims.L * sizeof(S);
    const int rows = (int)std::min<int64_t>(dar->dims.K, kStageBytes / kColsWaves / row);
    hipLaunchKernelGGL((k_chunk_adj_step<ST, S>), grid, dim3(64 * kColsWaves),
                       kColsWaves * rows * row, s, dar->pat(), dar->vals(), dc, cl, cs, ly, rows,
                       static_cast<const S*>(R), static_cast<S*>(Q), static_cast<S*>(A), st);
    return hipGetLastError();
  }
};

template <int ST, typename S>
struct RunApplyRows {
  static hipError_t run(const dode_dar* dar, const int32_t* dc, int32_t cl, const Layout& ly,
                        const void* Q, const void* X, void* out, double* part, int32_t n,
                        hipStream_t s) {
    dim3 grid(dar->dims.H, n);
    hipLaunchKernelGGL((k_apply_rows<ST, S>), grid, dim3(kRedBlock), 0, s, dar->pat(), dar->vals(),
                       dc, cl, ly, static_cast<const S*>(Q), static_cast<const S*>(X),
                       static_cast<S*>(out), part);
    return hipGetLastError();
  }
};

template <int ST, typename S>
struct RunAdjRows {
  static hipError_t run(const dode_dar* dar, const int32_t* dc, int32_t cl, const Layout& ly,
                        const void* R, void* G, int32_t n, hipStream_t s) {
    dim3 grid(dar->dims.T, n);
    hipLaunchKernelGGL((k_adjoint_rows<ST, S>), grid, dim3(kAdjBlock), 0, s, dar->pat(),
                       dar->vals(), dc, cl, ly, static_cast<const S*>(R), static_cast<S*>(G));
    return hipGetLastError();
  }
};

}  // namespace

hipError_t plain_chunk_resid(const dode_dar* dar, const int32_t* day_cluster, int32_t cluster,
                             const ChunkSched& cs, const Layout& ly, const void* Q, const void* X,
                             void* R, int32_t n_days, hipStream_t s) {
  return dispatch<RunResid>(dar, dar, day_cluster, cluster, cs, ly, Q, X, R, n_days, s);
}

hipError_t plain_chunk_adj_step(const dode_dar* dar, const int32_t* day_cluster, int32_t cluster,
                                const ChunkSched& cs, const Layout& ly, const void* R, void* Q,
                                void* A, int32_t n_days, const StepArgs& st, hipStream_t s) {
  return dispatch<RunAdjStep>(dar, dar, day_cluster, cluster, cs, ly, R, Q, A, n_days, st, s);
}

hipError_t plain_apply_rows(const dode_dar* dar, const int32_t* day_cluster, int32_t cluster,
                            const Layout& ly, const void* Q, const void* X, void* out, double* part,
                            int32_t n_days, hipStream_t s) {
  return dispatch<RunApplyRows>(dar, dar, day_cluster, cluster, ly, Q, X, out, part, n_days, s);
}

hipError_t plain_adjoint_rows(const dode_dar* dar, const int32_t* day_cluster, int32_t cluster,
                              const Layout& ly, const void* R, void* G, int32_t n_days,
                              hipStream_t s) {
  return dispatch<RunAdjRows>(dar, dar, day_cluster, cluster, ly, R, G, n_days, s);
}

namespace {

// Copies between the caller's days [D][rows][n] and the plan's state (Layout):
// plan entry (day i, row r, column k) at i*sd + r*sr + col_at(k, sb).  A lane
// moves four columns of one day; a wave 8 days x 8 such blocks, so it touches
// whole 128-byte lines on the caller's side and, in day-blocked rows, on the
// plan's side as well, with kCopyAhead of them in flight per lane.  A block
// takes 32 days of one row, and an XCD a contiguous range of (row, days): the
// lines two neighbouring blocks share meet in one L2.  Bound by memory: 1095 days
// of 500 links, 288 intervals, FP32 into day-blocked rows 599 -> 300 us (4.2
// TB/s), the demand of 150 ODs in 227 -> 102 us and back out 268 -> 96 us (one
// block per day and row, one column per thread, before: each line of the blocked
// rows was written by several XCDs).
constexpr int kCopyDays = 32, kCopyAhead = 4;

template <typename S>
struct Four {
  S v[4];
};
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));

// four columns from p on, zeros for the ones past `valid`
__device__ __forceinline__ Four<float> get_four(const float* p, int valid) {
  if (valid >= 4) {
    const f32x4u x = *reinterpret_cast<const f32x4u*>(p);
    return {{x[0], x[1], x[2], x[3]}};
  }
  return {{p[0], valid > 1 ? p[1] : 0.f, valid > 2 ? p[2] : 0.f, 0.f}};
}
__device__ __forceinline__ Four<double> get_four(const double* p, int valid) {
  if (valid >= 4) {
    const f64x2u x = *reinterpret_cast<const f64x2u*>(p), y = *reinterpret_cast<const f64x2u*>(p + 2);
    return {{x[0], x[1], y[0], y[1]}};
  }
  return {{p[0], valid > 1 ? p[1] : 0., valid > 2 ? p[2] : 0., 0.}};
}
__device__ __forceinline__ void put_four(float* p, const Four<float>& x, int valid) {
  if (valid >= 4) {
    *reinterpret_cast<f32x4u*>(p) = f32x4u{x.v[0], x.v[1], x.v[2], x.v[3]};
    return;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (k < valid) p[k] = x.v[k];
}
__device__ __forceinline__ void put_four(double* p, const Four<double>& x, int valid) {
  if (valid >= 4) {
    *reinterpret_cast<f64x2u*>(p) = f64x2u{x.v[0], x.v[1]};
    *reinterpret_cast<f64x2u*>(p + 2) = f64x2u{x.v[2], x.v[3]};
    return;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (k < valid) p[k] = x.v[k];
}

// Rows r0 .. r0+n_rows-1 of `rows`.  IN: caller to plan (with `clamp` projected onto
// >= 0), else plan to caller
template <typename S, bool IN>
__global__ void __launch_bounds__(256)
k_copy_days(const S* __restrict__ src, S* __restrict__ dst, const int32_t* __restrict__ order,
            int32_t D, int32_t rows, int32_t r0, int32_t n_rows, int32_t n, int64_t sd, int64_t sr,
            int64_t sb, int clamp) {
  const int tiles = (D + kCopyDays - 1) / kCopyDays;
  const int64_t n_blocks = (int64_t)n_rows * tiles, per = (n_blocks + 7) / 8;
  const int64_t b = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (b >= n_blocks || blockIdx.x / 8 >= per) return;
  const int row = (int)(b / tiles), r = r0 + row, tile = (int)(b - (int64_t)row * tiles);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = tile * kCopyDays + wave * 8 + (lane & 7);
  if (i >= D) return;
  const int64_t day = ((int64_t)order[i] * rows + r) * n, pos = i * sd + r * sr;
  const int nc = (n + 3) / 4;
  for (int c0 = lane >> 3; c0 < nc; c0 += 8 * kCopyAhead) {
    Four<S> x[kCopyAhead];
#pragma unroll
    for (int u = 0; u < kCopyAhead; ++u) {
      const int c = c0 + 8 * u;
      if (c < nc) x[u] = get_four(src + (IN ? day + 4 * c : pos + c * sb), n - 4 * c);
    }
#pragma unroll
    for (int u = 0; u < kCopyAhead; ++u) {
      const int c = c0 + 8 * u;
      if (c >= nc) continue;
      if (IN && clamp)
#pragma unroll
        for (int k = 0; k < 4; ++k) x[u].v[k] = x[u].v[k] > S(0) ? x[u].v[k] : S(0);
      put_four(dst + (IN ? pos + c * sb : day + 4 * c), x[u], n - 4 * c);
    }
  }
}

template <typename S, bool IN>
hipError_t copy_days(const void* src, void* dst, const int32_t* order, int32_t D, int32_t rows,
                     int32_t n, int64_t sd, int64_t sr, int64_t sb, bool clamp, hipStream_t s) {
  const int64_t tiles = (D + kCopyDays - 1) / kCopyDays;
  const int64_t most = (kGridThreads / 256 - 7) / tiles;   // rows of a launch
  if (most < 1) return hipErrorInvalidValue;
  for (int64_t r0 = 0; r0 < rows; r0 += most) {
    const int64_t nr = std::min<int64_t>(most, rows - r0);
    hipLaunchKernelGGL((k_copy_days<S, IN>), dim3((unsigned)((nr * tiles + 7) / 8 * 8)), dim3(256), 0, s,
                       static_cast<const S*>(src), static_cast<S*>(dst), order, D, rows, (int32_t)r0,
                       (int32_t)nr, n, sd, sr, sb, (int)clamp);
    if (const hipError_t e = hipGetLastError()) return e;
  }
  return hipSuccess;
}

template <typename S>
__global__ void k_zero(S* __restrict__ x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = S(0);
}

__global__ void k_set_counter(int32_t* c, int32_t v) { *c = v; }
__global__ void k_bump_counter(int32_t* c) { *c += 1; }

}  // namespace

hipError_t gather_rows(bool f64, const void* src, void* dst, const int32_t* order, int32_t D,
                       int32_t rows, int32_t n, int64_t sd, int64_t sr, int64_t sb, bool clamp,
                       hipStream_t s) {
  return f64 ? copy_days<double, true>(src, dst, order, D, rows, n, sd, sr, sb, clamp, s)
             : copy_days<float, true>(src, dst, order, D, rows, n, sd, sr, sb, clamp, s);
}

hipError_t scatter_rows(bool f64, const void* src, void* dst, const int32_t* order, int32_t D,
                        int32_t rows, int32_t n, int64_t sd, int64_t sr, int64_t sb, hipStream_t s) {
  return f64 ? copy_days<double, false>(src, dst, order, D, rows, n, sd, sr, sb, false, s)
             : copy_days<float, false>(src, dst, order, D, rows, n, sd, sr, sb, false, s);
}

hipError_t fill_zero(bool f64, void* x, int64_t n, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>(4096, std::max<int64_t>(1, (n + 255) / 256));
  if (f64)
    hipLaunchKernelGGL(k_zero<double>, dim3(blocks), dim3(256), 0, s, static_cast<double*>(x), n);
  else
    hipLaunchKernelGGL(k_zero<float>, dim3(blocks), dim3(256), 0, s, static_cast<float*>(x), n);
  return hipGetLastError();
}

hipError_t set_counter(int32_t* c, int32_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(1), 0, s, c, v);
  return hipGetLastError();
}

hipError_t bump_counter(int32_t* c, hipStream_t s) {
  hipLaunchKernelGGL(k_bump_counter, dim3(1), dim3(1), 0, s, c);
  return hipGetLastError();
}

hipError_t sum_partials(const double* part, int32_t n_per, int32_t n_days, double* out,
                        hipStream_t s, const int32_t* order) {
  hipLaunchKernelGGL(k_sum_partials, dim3((n_days + 3) / 4), dim3(kRedBlock), 0, s, part, n_per,
                     n_days, out, order);
  return hipGetLastError();
}

hipError_t max_partials(const double* part, int32_t n_per, int32_t n_days, double* out,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_max_partials, dim3((n_days + 3) / 4), dim3(kRedBlock), 0, s, part, n_per,
                     n_days, out);
  return hipGetLastError();
}

hipError_t kkt_partials(bool f64, const void* Q, const void* G, int32_t T, int32_t P,
                        int32_t n_days, double* part, hipStream_t s) {
  if (f64)
    hipLaunchKernelGGL(k_kkt_partials<double>, dim3((T + 3) / 4, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const double*>(Q), static_cast<const double*>(G), T, P, part);
  else
    hipLaunchKernelGGL(k_kkt_partials<float>, dim3((T + 3) / 4, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const float*>(Q), static_cast<const float*>(G), T, P, part);
  return hipGetLastError();
}

hipError_t x_moment_partials(bool f64, const void* X, int32_t H, int32_t L, int32_t n_days,
                             const double* sum_x, double* part, hipStream_t s) {
  if (f64)
    hipLaunchKernelGGL(k_x_moment<double>, dim3((H + 3) / 4, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const double*>(X), H, L, sum_x, part);
  else
    hipLaunchKernelGGL(k_x_moment<float>, dim3((H + 3) / 4, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const float*>(X), H, L, sum_x, part);
  return hipGetLastError();
}

hipError_t r2_finish(const double* loss, const double* sst, int32_t n_days, double* r2,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_r2, dim3((n_days + 127) / 128), dim3(128), 0, s, loss, sst, n_days, r2);
  return hipGetLastError();
}

hipError_t check_finite(bool f64, const void* X, int64_t n, int32_t* flag, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>(4096, (n + 255) / 256 > 0 ? (n + 255) / 256 : 1);
  if (f64)
    hipLaunchKernelGGL(k_check_finite<double>, dim3(blocks), dim3(256), 0, s,
                       static_cast<const double*>(X), n, flag);
  else
    hipLaunchKernelGGL(k_check_finite<float>, dim3(blocks), dim3(256), 0, s,
                       static_cast<const float*>(X), n, flag);
  return hipGetLastError();
}

hipError_t clamp_nonneg(bool f64, void* Q, int64_t n, hipStream_t s) {
  const int64_t blocks = std::min<int64_t>(4096, (n + 255) / 256 > 0 ? (n + 255) / 256 : 1);
  if (f64)
    hipLaunchKernelGGL(k_clamp<double>, dim3(blocks), dim3(256), 0, s, static_cast<double*>(Q), n);
  else
    hipLaunchKernelGGL(k_clamp<float>, dim3(blocks), dim3(256), 0, s, static_cast<float*>(Q), n);
  return hipGetLastError();
}
