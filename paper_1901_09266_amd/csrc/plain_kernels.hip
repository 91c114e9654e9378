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

#include <cmath>

namespace {

constexpr int kRowsBlock = 256;
constexpr int kColsBlock = 64;
constexpr int kRedBlock = 256;
constexpr size_t kQStageBytes = 32768;   // demand rows staged in LDS by the forward

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

__device__ double block_max(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int w = kRedBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + w]);
    __syncthreads();
  }
  return sh[0];
}

// ------------------------------------------------------------- kernels --
// With STAGE the block first copies the K demand rows its links read,
// Q_d[h-l] for l < K, into LDS (row l at l*P; rows outside the day are
// zeros that no lane reads), so the walk's demand gathers are LDS reads.
template <int ST, typename S, bool STAGE>
__global__ void __launch_bounds__(kRowsBlock)
k_chunk_resid(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, ChunkSched cs,
              Layout ly, const S* __restrict__ Q, const S* __restrict__ X, S* __restrict__ R) {
  extern __shared__ unsigned char q_stage[];
  const int a = blockIdx.x * kRowsBlock + threadIdx.x;
  const int s = blockIdx.y, d = blockIdx.z;
  cs = resolve_epoch(cs);
  const int c = day_cl(day_cluster, cluster, d);
  if (cs.j0 + s >= pt.H) return;   // the whole block
  const int h = cs.perm[c * pt.H + cs.j0 + s];
  S xhat;
  if constexpr (STAGE) {
    S* qs = reinterpret_cast<S*>(q_stage);
    const S* qd = Q + d * ly.q_d;
    for (int i = threadIdx.x; i < pt.K * pt.P; i += kRowsBlock) {
      const int l = i / pt.P, p = i % pt.P, t = h - l;
      qs[i] = (t >= 0 && t < pt.T) ? qd[(int64_t)t * ly.q_t + col_at(p, ly.q_b)] : S(0);
    }
    __syncthreads();
    if (a >= pt.L) return;
    // row t = h - l of the staged copy sits at (h - t) * P: base h*P, stride -P
    xhat = row_dot<ST, S>(pt, v, c, h, a, qs + (int64_t)h * pt.P, -(int64_t)pt.P, 4);
  } else {
    if (a >= pt.L) return;
    xhat = row_dot<ST, S>(pt, v, c, h, a, Q + d * ly.q_d, ly.q_t, ly.q_b);
  }
  R[d * ly.r_d + s * ly.r_s + col_at(a, ly.r_b)] = xhat - X[d * ly.x_d + h * ly.x_h + col_at(a, ly.x_b)];
}

template <int ST, typename S>
__global__ void __launch_bounds__(kColsBlock)
k_chunk_adj_step(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, ChunkSched cs,
                 Layout ly, const S* __restrict__ R, S* __restrict__ Q, S* __restrict__ A,
                 StepArgs st) {
  const int p = blockIdx.x * kColsBlock + threadIdx.x;
  const int i = blockIdx.y, d = blockIdx.z;
  if (p >= pt.P) return;
  cs = resolve_epoch(cs);
  const int c = day_cl(day_cluster, cluster, d);
  const int t = cs.touched[((int64_t)c * cs.max_touched + i) * desc_width(pt.K) + kDescT];
  if (t < 0) return;
  const S g = col_dot_chunk<ST, S>(pt, v, c, t, p, cs.pos + (int64_t)c * pt.H, cs.j0, cs.bh,
                                   R + d * ly.r_d, ly.r_s, ly.r_b);
  const int64_t idx = d * ly.q_d + t * ly.q_t + col_at(p, ly.q_b);
  S q = Q[idx];
  if (st.optimizer == 0) {
    const S acc = A[idx] + g * g;
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

template <int ST, typename S>
__global__ void __launch_bounds__(kColsBlock)
k_adjoint_rows(DevPat pt, DevVals v, const int32_t* day_cluster, int32_t cluster, Layout ly,
               const S* __restrict__ R, S* __restrict__ G) {
  const int t = blockIdx.x, d = blockIdx.y;
  const int c = day_cl(day_cluster, cluster, d);
  const S* Rd = R + d * ly.r_d;
  for (int p = threadIdx.x; p < pt.P; p += kColsBlock)
    G[d * ly.q_d + t * ly.q_t + col_at(p, ly.q_b)] =
        col_dot_chunk<ST, S>(pt, v, c, t, p, nullptr, 0, pt.H, Rd, ly.r_s, ly.r_b);
}

// One wave per day: lane i takes partials i, i+64, ..., then a butterfly (fixed
// order).  One thread per day left a serial chain of 288 loads: 22 us for any
// number of days.
__global__ void __launch_bounds__(kRedBlock)
k_sum_partials(const double* __restrict__ part, int32_t n_per, int32_t n_days,
               double* __restrict__ out) {
  const int d = blockIdx.x * (kRedBlock / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (d >= n_days) return;
  double s = 0.0;
  for (int i = lane; i < n_per; i += 64) s += part[(int64_t)d * n_per + i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) out[d] = s;
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

template <typename S>
__global__ void __launch_bounds__(kRedBlock)
k_kkt_partials(const S* __restrict__ Q, const S* __restrict__ G, int32_t T, int32_t P,
               double* __restrict__ part) {
  __shared__ double sh[kRedBlock];
  const int t = blockIdx.x, d = blockIdx.y;
  double m = 0.0;
  for (int p = threadIdx.x; p < P; p += kRedBlock) {
    const int64_t i = ((int64_t)d * T + t) * P + p;
    const double q = Q[i], g = G[i];
    m = fmax(m, fabs(q < g ? q : g));
  }
  const double r = block_max(m, sh);
  if (threadIdx.x == 0) part[(int64_t)d * T + t] = r;
}

// First pass (sum_x == nullptr): per (d, h) sum of x.  Second pass: sum of (x - mean)^2.
template <typename S>
__global__ void __launch_bounds__(kRedBlock)
k_x_moment(const S* __restrict__ X, int32_t H, int32_t L, const double* __restrict__ sum_x,
           double* __restrict__ part) {
  __shared__ double sh[kRedBlock];
  const int h = blockIdx.x, d = blockIdx.y;
  const double mean = sum_x ? sum_x[d] / (static_cast<double>(H) * L) : 0.0;
  double s = 0.0;
  for (int a = threadIdx.x; a < L; a += kRedBlock) {
    const double x = X[((int64_t)d * H + h) * L + a];
    s += sum_x ? (x - mean) * (x - mean) : x;
  }
  const double r = block_sum(s, sh);
  if (threadIdx.x == 0) part[(int64_t)d * H + h] = r;
}

__global__ void k_r2(const double* loss, const double* sst, int32_t n, double* r2) {
  const int d = blockIdx.x * blockDim.x + threadIdx.x;
  if (d < n) r2[d] = 1.0 - loss[d] / sst[d];
}

template <typename S>
__global__ void k_check_finite(const S* __restrict__ X, int64_t n, int32_t* flag) {
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    bad |= !isfinite(X[i]);
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
    if (stage <= kQStageBytes)
      hipLaunchKernelGGL((k_chunk_resid<ST, S, true>), grid, dim3(kRowsBlock), stage, s, dar->pat(),
                         dar->vals(), dc, cl, cs, ly, static_cast<const S*>(Q),
                         static_cast<const S*>(X), static_cast<S*>(R));
    else
      hipLaunchKernelGGL((k_chunk_resid<ST, S, false>), grid, dim3(kRowsBlock), 0, s, dar->pat(),
                         dar->vals(), dc, cl, cs, ly, static_cast<const S*>(Q),
                         static_cast<const S*>(X), static_cast<S*>(R));
    return hipGetLastError();
  }
};

template <int ST, typename S>
struct RunAdjStep {
  static hipError_t run(const dode_dar* dar, const int32_t* dc, int32_t cl, const ChunkSched& cs,
                        const Layout& ly, const void* R, void* Q, void* A, int32_t n,
                        const StepArgs& st, hipStream_t s) {
    dim3 grid((dar->dims.P + kColsBlock - 1) / kColsBlock, cs.max_touched, n);
    hipLaunchKernelGGL((k_chunk_adj_step<ST, S>), grid, dim3(kColsBlock), 0, s, dar->pat(),
                       dar->vals(), dc, cl, cs, ly, static_cast<const S*>(R), static_cast<S*>(Q),
                       static_cast<S*>(A), st);
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
    hipLaunchKernelGGL((k_adjoint_rows<ST, S>), grid, dim3(kColsBlock), 0, s, dar->pat(),
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

// dst[r][i][k] = src[order[i]][r][k]; block (i, r), threads over k.
template <typename S>
__global__ void k_gather(const S* __restrict__ src, S* __restrict__ dst, const int32_t* order,
                         int32_t rows, int32_t n, int64_t sd, int64_t sr, int64_t sb, int clamp) {
  const int i = blockIdx.x, r = blockIdx.y;
  const S* a = src + ((int64_t)order[i] * rows + r) * n;
  S* b = dst + (int64_t)i * sd + (int64_t)r * sr;
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    const S v = a[k];
    b[col_at(k, sb)] = clamp ? (v > S(0) ? v : S(0)) : v;
  }
}

template <typename S>
__global__ void k_scatter(const S* __restrict__ src, S* __restrict__ dst, const int32_t* order,
                          int32_t rows, int32_t n, int64_t sd, int64_t sr, int64_t sb) {
  const int i = blockIdx.x, r = blockIdx.y;
  const S* a = src + (int64_t)i * sd + (int64_t)r * sr;
  S* b = dst + ((int64_t)order[i] * rows + r) * n;
  for (int k = threadIdx.x; k < n; k += blockDim.x) b[k] = a[col_at(k, sb)];
}

template <typename S>
__global__ void k_zero(S* __restrict__ x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = S(0);
}

__global__ void k_set_counter(int32_t* c, int32_t v) { *c = v; }
__global__ void k_bump_counter(int32_t* c) { *c += 1; }

__global__ void k_permute_loss(const double* __restrict__ src, const int32_t* __restrict__ order,
                               int32_t D, double* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < D) dst[order[i]] = src[i];
}

}  // namespace

hipError_t gather_rows(bool f64, const void* src, void* dst, const int32_t* order, int32_t D,
                       int32_t rows, int32_t n, int64_t sd, int64_t sr, int64_t sb, bool clamp,
                       hipStream_t s) {
  const dim3 grid(D, rows);
  if (f64)
    hipLaunchKernelGGL(k_gather<double>, grid, dim3(256), 0, s, static_cast<const double*>(src),
                       static_cast<double*>(dst), order, rows, n, sd, sr, sb, (int)clamp);
  else
    hipLaunchKernelGGL(k_gather<float>, grid, dim3(256), 0, s, static_cast<const float*>(src),
                       static_cast<float*>(dst), order, rows, n, sd, sr, sb, (int)clamp);
  return hipGetLastError();
}

hipError_t scatter_rows(bool f64, const void* src, void* dst, const int32_t* order, int32_t D,
                        int32_t rows, int32_t n, int64_t sd, int64_t sr, int64_t sb, hipStream_t s) {
  const dim3 grid(D, rows);
  if (f64)
    hipLaunchKernelGGL(k_scatter<double>, grid, dim3(256), 0, s, static_cast<const double*>(src),
                       static_cast<double*>(dst), order, rows, n, sd, sr, sb);
  else
    hipLaunchKernelGGL(k_scatter<float>, grid, dim3(256), 0, s, static_cast<const float*>(src),
                       static_cast<float*>(dst), order, rows, n, sd, sr, sb);
  return hipGetLastError();
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

hipError_t permute_loss(const double* src, const int32_t* order, int32_t D, double* dst,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_permute_loss, dim3((D + 255) / 256), dim3(256), 0, s, src, order, D, dst);
  return hipGetLastError();
}

hipError_t sum_partials(const double* part, int32_t n_per, int32_t n_days, double* out,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_sum_partials, dim3((n_days + 3) / 4), dim3(kRedBlock), 0, s, part, n_per,
                     n_days, out);
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
    hipLaunchKernelGGL(k_kkt_partials<double>, dim3(T, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const double*>(Q), static_cast<const double*>(G), T, P, part);
  else
    hipLaunchKernelGGL(k_kkt_partials<float>, dim3(T, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const float*>(Q), static_cast<const float*>(G), T, P, part);
  return hipGetLastError();
}

hipError_t x_moment_partials(bool f64, const void* X, int32_t H, int32_t L, int32_t n_days,
                             const double* sum_x, double* part, hipStream_t s) {
  if (f64)
    hipLaunchKernelGGL(k_x_moment<double>, dim3(H, n_days), dim3(kRedBlock), 0, s,
                       static_cast<const double*>(X), H, L, sum_x, part);
  else
    hipLaunchKernelGGL(k_x_moment<float>, dim3(H, n_days), dim3(kRedBlock), 0, s,
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
