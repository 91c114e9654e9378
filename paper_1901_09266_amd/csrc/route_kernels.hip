// Route-choice kernels: the assignment matrix from route portions (eqs.
// "logit", "rt", "flow", "assign"), with portions from free logits per path or
// from the mean path costs of a pattern, and the loss gradient with respect to
// the assignment values and the free logits.  One thread or block per output
// entry, fixed summation order, FP64 accumulation for the reductions.
#include "dode_internal.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int kBlock = 256;

__device__ double block_sum256(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Per row t < n_rows and OD p: pi[t][k] = exp(a z[t][k] - max) / sum over the
// paths of OD p (FP64); one thread per (t, p).  z rows are zs apart (zs = 0
// repeats one row); a = 1 for free logits, -theta for costs.  When pi_out is
// set the portions are also written there in the storage type.
template <typename S>
__global__ void k_softmax(DevRoutes r, int32_t n_rows, const S* __restrict__ z, int64_t zs,
                          double a, double* __restrict__ pi, S* __restrict__ pi_out) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n_rows * r.P) return;
  const int32_t t = (int32_t)(idx / r.P), p = (int32_t)(idx % r.P);
  const S* zt = z + t * zs;
  double* pt = pi + (int64_t)t * r.n_paths;
  const int k0 = r.od_ptr[p], k1 = r.od_ptr[p + 1];
  double zmax = -INFINITY;
  for (int i = k0; i < k1; ++i) zmax = fmax(zmax, a * static_cast<double>(zt[r.od_paths[i]]));
  double s = 0.0;
  for (int i = k0; i < k1; ++i) s += exp(a * static_cast<double>(zt[r.od_paths[i]]) - zmax);
  for (int i = k0; i < k1; ++i) {
    const int k = r.od_paths[i];
    const double v = exp(a * static_cast<double>(zt[k]) - zmax) / s;
    pt[k] = v;
    if (pi_out) pi_out[(int64_t)t * r.n_paths + k] = static_cast<S>(v);
  }
}

// W[l][t][nz] = sum over pairs m feeding nz of Rr[l][t][m] * pi[t][path(m)]
// (eq. "assign"); pi rows are ps apart (ps = 0: portions that do not depend
// on the interval).  Pairs are summed in increasing order.
// A thread takes one entry of kRhoRows blocks (l, t): the lists are read once
// for all of them and their ratios are in flight together (6000 entries, 288
// intervals, 6 lags: 89.7 -> 58.7 us with a thread and two 64-bit divisions per
// value before).
constexpr int kRhoRows = 8;
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_rho_from_pi(DevRoutes r, const S* __restrict__ Rr, const double* __restrict__ pi, int64_t ps,
              S* __restrict__ W) {
  const int64_t nz = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (nz >= r.nnz) return;
  const int n_lt = r.K * r.T;
  for (int lt0 = blockIdx.y * kRhoRows; lt0 < n_lt; lt0 += gridDim.y * kRhoRows) {
    double s[kRhoRows];
#pragma unroll
    for (int u = 0; u < kRhoRows; ++u) s[u] = 0.0;
    for (int i = r.nz_ptr[nz]; i < r.nz_ptr[nz + 1]; ++i) {
      const int m = r.nz_pairs[i], k = r.pair_path[m];
      S x[kRhoRows];
      double p[kRhoRows];
#pragma unroll
      for (int u = 0; u < kRhoRows; ++u) {
        const int lt = min(lt0 + u, n_lt - 1);
        x[u] = Rr[(int64_t)lt * r.n_pairs + m];
        p[u] = pi[(lt % r.T) * ps + k];
      }
#pragma unroll
      for (int u = 0; u < kRhoRows; ++u) s[u] += static_cast<double>(x[u]) * p[u];
    }
#pragma unroll
    for (int u = 0; u < kRhoRows; ++u)
      if (lt0 + u < n_lt) W[(int64_t)(lt0 + u) * r.nnz + nz] = static_cast<S>(s[u]);
  }
}

// dpi_k = sum_{lt, pairs m of k} Rr[lt][m] dW[lt][pair_nz[m]]; one block per path,
// thread i takes terms i, i + 256, ... (four in flight; their block and pair are
// stepped, not divided out: 114 -> 106 us for 450 routes, 288 intervals, 6 lags).
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_dpi(DevRoutes r, const S* __restrict__ Rr, const S* __restrict__ dW, double* __restrict__ dpi) {
  __shared__ double sh[kBlock];
  constexpr int U = 4;
  const int k = blockIdx.x;
  const int m0 = r.pair_ptr[k], per = r.pair_ptr[k + 1] - m0;
  const int n_lt = r.K * r.T;
  double s = 0.0;
  if (per > 0) {
    int lt = threadIdx.x / per, j = threadIdx.x % per;
    const int dl = kBlock / per, dj = kBlock % per;
    while (lt < n_lt) {
      S x[U], w[U];
      bool in[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        in[u] = lt < n_lt;
        const int64_t at = min(lt, n_lt - 1);
        x[u] = Rr[at * r.n_pairs + m0 + j];
        w[u] = dW[at * r.nnz + r.pair_nz[m0 + j]];
        lt += dl;
        j += dj;
        if (j >= per) {
          j -= per;
          ++lt;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (in[u]) s += static_cast<double>(x[u]) * static_cast<double>(w[u]);
    }
  }
  const double tot = block_sum256(s, sh);
  if (threadIdx.x == 0) dpi[k] = tot;
}

// dz_k = pi_k (dpi_k - sum_{k' serving od(k)} pi_k' dpi_k'); one thread per path.
template <typename S>
__global__ void k_dz(DevRoutes r, const double* __restrict__ pi, const double* __restrict__ dpi,
                     S* __restrict__ dz) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= r.n_paths) return;
  const int p = r.path_od[k];
  double s = 0.0;
  for (int i = r.od_ptr[p]; i < r.od_ptr[p + 1]; ++i) {
    const int k2 = r.od_paths[i];
    s += pi[k2] * dpi[k2];
  }
  dz[k] = static_cast<S>(pi[k] * (dpi[k] - s));
}

// dW[l][t][nz(a,p)] = scale * sum_d R[d][t+l][a] Q[d][t][p]   (0 where t+l >= H).
template <typename S>
__global__ void k_dW(DevPat pt, const int32_t* __restrict__ row_of_nz, const S* __restrict__ R,
                     const S* __restrict__ Q, int32_t n_days, double scale, S* __restrict__ dW) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)pt.K * pt.T * pt.nnz;
  if (idx >= total) return;
  const int64_t lt = idx / pt.nnz, nz = idx % pt.nnz;
  const int l = (int)(lt / pt.T), t = (int)(lt % pt.T);
  double s = 0.0;
  if (t + l < pt.H) {
    const int a = row_of_nz[nz], p = pt.col[nz];
    for (int d = 0; d < n_days; ++d)
      s += static_cast<double>(R[((int64_t)d * pt.H + t + l) * pt.L + a]) *
           static_cast<double>(Q[((int64_t)d * pt.T + t) * pt.P + p]);
  }
  dW[idx] = static_cast<S>(scale * s);
}

// The same with the day rows of one (l, t) staged in LDS, kDwDays days at a time
// (line a's days next to each other: two 16-byte reads per side and entry), each
// thread kDwEntries entries.  One thread per value read every residual and demand
// from memory at its own address: 254 -> 149 us for 30 days of 6000 entries, 288
// intervals, 6 lags.  Each value's sum runs over the days in order, as above.
constexpr int kDwDays = 8, kDwEntries = 12;
constexpr int64_t kDwLds = 65536;
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_dW_staged(DevPat pt, const int32_t* __restrict__ row_of_nz, const S* __restrict__ R,
            const S* __restrict__ Q, int32_t n_days, double scale, S* __restrict__ dW) {
  extern __shared__ __align__(16) unsigned char dw_stage[];
  S* rs = reinterpret_cast<S*>(dw_stage);
  S* qs = rs + (int64_t)pt.L * kDwDays;
  const int t = blockIdx.y, l = blockIdx.z;
  const int64_t nz0 = (int64_t)blockIdx.x * kBlock * kDwEntries + threadIdx.x;
  S* out = dW + ((int64_t)l * pt.T + t) * pt.nnz;
  double s[kDwEntries];
  int a[kDwEntries], p[kDwEntries];
#pragma unroll
  for (int u = 0; u < kDwEntries; ++u) {
    const int64_t nz = min(nz0 + (int64_t)u * kBlock, pt.nnz - 1);
    s[u] = 0.0;
    a[u] = row_of_nz[nz] * kDwDays;
    p[u] = pt.col[nz] * kDwDays;
  }
  const int days = t + l < pt.H ? n_days : 0;
  for (int d0 = 0; d0 < days; d0 += kDwDays) {
    if (d0 > 0) __syncthreads();
    auto stage = [&](const S* src, int64_t day, int n, S* to) {
      for (int i = threadIdx.x; i < n; i += kBlock) {
        S x[kDwDays];
#pragma unroll
        for (int d = 0; d < kDwDays; ++d)
          x[d] = src[(int64_t)min(d0 + d, days - 1) * day + i];
#pragma unroll
        for (int d = 0; d < kDwDays; ++d) to[i * kDwDays + d] = x[d];
      }
    };
    stage(R + (int64_t)(t + l) * pt.L, (int64_t)pt.H * pt.L, pt.L, rs);
    stage(Q + (int64_t)t * pt.P, (int64_t)pt.T * pt.P, pt.P, qs);
    __syncthreads();
    const int nd = min(kDwDays, days - d0);
#pragma unroll
    for (int u = 0; u < kDwEntries; ++u) {
      if (nz0 - threadIdx.x + (int64_t)u * kBlock >= pt.nnz) break;
#pragma unroll
      for (int d = 0; d < kDwDays; ++d) {
        if (d >= nd) break;
        s[u] += static_cast<double>(rs[a[u] + d]) * static_cast<double>(qs[p[u] + d]);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < kDwEntries; ++u)
    if (nz0 + (int64_t)u * kBlock < pt.nnz) out[nz0 + (int64_t)u * kBlock] = static_cast<S>(scale * s[u]);
}

template <typename S>
__global__ void k_scale(S* __restrict__ x, int64_t n, double f) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = static_cast<S>(static_cast<double>(x[i]) * f);
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

template <typename S>
void launch_rho(const DevRoutes& r, int32_t n_rows, const S* Rr, const S* z, int64_t zs, double a,
                double* pi, S* pi_out, S* W, hipStream_t s) {
  hipLaunchKernelGGL(k_softmax<S>, dim3(blocks_for((int64_t)n_rows * r.P)), dim3(kBlock), 0, s, r,
                     n_rows, z, zs, a, pi, pi_out);
  const dim3 grid(blocks_for(r.nnz), (unsigned)std::min((r.K * r.T + kRhoRows - 1) / kRhoRows, 65535));
  hipLaunchKernelGGL(k_rho_from_pi<S>, grid, dim3(kBlock), 0, s, r, Rr, pi,
                     n_rows > 1 ? (int64_t)r.n_paths : 0, W);
}

template <typename S>
hipError_t launch_dW(const dode_dar* dar, const void* R, const void* Q, int32_t n_days, double scale,
                     void* dW, hipStream_t s) {
  const dode_dims& dm = dar->dims;
  auto go = [&](auto kern, dim3 grid, size_t lds) {
    hipLaunchKernelGGL(kern, grid, dim3(kBlock), lds, s, dar->pat(), dar->d_row_of_nz,
                       static_cast<const S*>(R), static_cast<const S*>(Q), n_days, scale,
                       static_cast<S*>(dW));
  };
  const int64_t lds = ((int64_t)dm.L + dm.P) * kDwDays * sizeof(S);
  const int64_t tiles = (dar->nnz + kBlock * kDwEntries - 1) / (kBlock * kDwEntries);
  if (lds <= kDwLds && dm.T <= 65535)
    go(k_dW_staged<S>, dim3((unsigned)tiles, dm.T, dm.K), lds);
  else   // rows too long to stage
    go(k_dW<S>, dim3(blocks_for((int64_t)dm.K * dm.T * dar->nnz)), 0);
  return hipGetLastError();
}

}  // namespace

hipError_t routes_rho(const DevRoutes& r, bool f64, const void* Rr, const void* z, void* W,
                      double* pi, hipStream_t s) {
  if (f64)
    launch_rho<double>(r, 1, static_cast<const double*>(Rr), static_cast<const double*>(z), 0, 1.0,
                       pi, nullptr, static_cast<double*>(W), s);
  else
    launch_rho<float>(r, 1, static_cast<const float*>(Rr), static_cast<const float*>(z), 0, 1.0, pi,
                      nullptr, static_cast<float*>(W), s);
  return hipGetLastError();
}

hipError_t routes_rho_costs(const DevRoutes& r, bool f64, const void* Rr, const void* cost,
                            double theta, void* portions, void* W, double* pi, hipStream_t s) {
  if (f64)
    launch_rho<double>(r, r.T, static_cast<const double*>(Rr), static_cast<const double*>(cost),
                       r.n_paths, -theta, pi, static_cast<double*>(portions),
                       static_cast<double*>(W), s);
  else
    launch_rho<float>(r, r.T, static_cast<const float*>(Rr), static_cast<const float*>(cost),
                      r.n_paths, -theta, pi, static_cast<float*>(portions), static_cast<float*>(W),
                      s);
  return hipGetLastError();
}

hipError_t routes_logits_bwd(const DevRoutes& r, bool f64, const void* Rr, const void* z,
                             const void* dW, void* dz, double* pi, double* dpi, hipStream_t s) {
  if (f64) {
    hipLaunchKernelGGL(k_softmax<double>, dim3(blocks_for(r.P)), dim3(kBlock), 0, s, r, 1,
                       static_cast<const double*>(z), (int64_t)0, 1.0, pi, (double*)nullptr);
    hipLaunchKernelGGL(k_dpi<double>, dim3(r.n_paths), dim3(kBlock), 0, s, r,
                       static_cast<const double*>(Rr), static_cast<const double*>(dW), dpi);
    hipLaunchKernelGGL(k_dz<double>, dim3(blocks_for(r.n_paths)), dim3(kBlock), 0, s, r, pi, dpi,
                       static_cast<double*>(dz));
  } else {
    hipLaunchKernelGGL(k_softmax<float>, dim3(blocks_for(r.P)), dim3(kBlock), 0, s, r, 1,
                       static_cast<const float*>(z), (int64_t)0, 1.0, pi, (float*)nullptr);
    hipLaunchKernelGGL(k_dpi<float>, dim3(r.n_paths), dim3(kBlock), 0, s, r,
                       static_cast<const float*>(Rr), static_cast<const float*>(dW), dpi);
    hipLaunchKernelGGL(k_dz<float>, dim3(blocks_for(r.n_paths)), dim3(kBlock), 0, s, r, pi, dpi,
                       static_cast<float*>(dz));
  }
  return hipGetLastError();
}

hipError_t loss_bwd_dW(const dode_dar* dar, const void* R, const void* Q, int32_t n_days,
                       double scale, void* dW, hipStream_t s) {
  return is_f64(dar) ? launch_dW<double>(dar, R, Q, n_days, scale, dW, s)
                     : launch_dW<float>(dar, R, Q, n_days, scale, dW, s);
}

hipError_t scale_state(bool f64, void* x, int64_t n, double f, hipStream_t s) {
  const unsigned b = (unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, blocks_for(n)));
  if (f64)
    hipLaunchKernelGGL(k_scale<double>, dim3(b), dim3(kBlock), 0, s, static_cast<double*>(x), n, f);
  else
    hipLaunchKernelGGL(k_scale<float>, dim3(b), dim3(kBlock), 0, s, static_cast<float*>(x), n, f);
  return hipGetLastError();
}
