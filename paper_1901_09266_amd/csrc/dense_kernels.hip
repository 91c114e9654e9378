// Algorithm 1 on a dense B [m][n] (section "Solution algorithm"), the
// workload of the efficiency experiment (section "Algorithm efficiency").
//
// A minibatch of rows o = perm[s0 .. s0+nr) takes three launches, all
// HBM-bound on B (each row of the minibatch is streamed twice):
//   k_dense_resid    one wave per minibatch row: r[s] = B[o_s] . q - y[o_s];
//                    lanes read 16-byte vectors across the row and the wave
//                    sums them with a butterfly reduction;
//   k_dense_colsum   split-K adjoint: block (column block, slice of kSliceRows
//                    rows) writes part[slice][j] = sum over its rows of
//                    B[o_s][j] r[s], four consecutive columns per lane, so a
//                    wave reads 1 KiB of one row per step; the block's four
//                    waves split the slice's rows and meet in LDS;
//   k_dense_update   one block per 16 columns: g = the slices' partial sums
//                    (FP64, 16 lane groups over the slices, added in a fixed
//                    order), then Adagrad (or a fixed step) and the
//                    projection q = max(q, 0).
// The epoch loss ||B q - y||^2 (optional) uses the residual kernel over all
// rows in natural order, and FP64 sums in a fixed order, one block per epoch for
// as many epochs as the scratch holds.  Where one minibatch holds every row its
// residuals are those of the loss before it (same rows, same q), so such an
// epoch streams B twice instead of three times: with losses n = 500 takes 612
// instead of 883 us for 50 epochs, n = 1525 in FP64 488 instead of 926 us for 18.
// B may also be stored as bf16 (FP32 arithmetic and state): the *_bf16
// kernels read 16 bytes = 8 values per lane and load.
#include "dode_internal.h"

#include <algorithm>

namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;
constexpr int kSliceRows = 128;
constexpr int kRowsAhead = 8;   // rows in flight per wave (column sums)

template <typename S>
struct Vec;
template <>
struct Vec<float> {
  using T = float4;
  static constexpr int N = 4;
};
template <>
struct Vec<double> {
  using T = double2;
  static constexpr int N = 2;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// r[s] = B[row] . q - y[row] for rows[s], s < nr (rows == nullptr: row s).
// VEC: rows are 16-byte aligned and n is a multiple of the vector width.
template <typename S, bool VEC>
__global__ void __launch_bounds__(kBlock)
k_dense_resid(int32_t n, int32_t nr, const int32_t* __restrict__ rows, const S* __restrict__ B,
              const S* __restrict__ y, const S* __restrict__ q, S* __restrict__ r) {
  const int s = blockIdx.x * kWaves + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (s >= nr) return;
  const int32_t i = rows ? rows[s] : s;
  const S* row = B + (int64_t)i * n;
  S acc = S(0);
  if (VEC) {
    using V = typename Vec<S>::T;
    constexpr int W = Vec<S>::N;
    const V* rv = reinterpret_cast<const V*>(row);
    const V* qv = reinterpret_cast<const V*>(q);
    const int nv = n / W;
    S a2 = S(0);
    int j = lane;
    for (; j + 64 < nv; j += 128) {   // two vectors in flight per lane
      const V b0 = rv[j], b1 = rv[j + 64], q0 = qv[j], q1 = qv[j + 64];
      if constexpr (W == 4) {
        acc += b0.x * q0.x + b0.y * q0.y + b0.z * q0.z + b0.w * q0.w;
        a2 += b1.x * q1.x + b1.y * q1.y + b1.z * q1.z + b1.w * q1.w;
      } else {
        acc += b0.x * q0.x + b0.y * q0.y;
        a2 += b1.x * q1.x + b1.y * q1.y;
      }
    }
    if (j < nv) {
      const V b0 = rv[j], q0 = qv[j];
      if constexpr (W == 4)
        acc += b0.x * q0.x + b0.y * q0.y + b0.z * q0.z + b0.w * q0.w;
      else
        acc += b0.x * q0.x + b0.y * q0.y;
    }
    acc += a2;
  } else {
    for (int j = lane; j < n; j += 64) acc += row[j] * q[j];
  }
  acc = wave_sum(acc);
  if (lane == 0) r[s] = acc - y[i];
}

// The rows of one slice and their residuals (residual of slot s: r[s], or
// r[row] when they are kept by row).  With LDS they are read once per block, so
// the loads of B depend on nothing and kRowsAhead rows are in flight per wave:
// 4.1 against 4.8 us for 500 x 500, where a block has only its own latency to
// wait for.  A grid that fills the chip several times hides the two loads
// before each row, and pays for the block's first barrier: 23.7 against 24.5 us
// for 6000 x 6000.  The line lies at two blocks per CU, for FP64 (half the
// columns per block) at one; 20 epochs with and without LDS: FP32 n = 1500 (72
// blocks) 306 and 345 us, 4000 (512) 585 and 595; FP64 1500 (144) 348 and 379,
// 2300 (324) 501 and 498, 4000 (1024) 943 and 934; bf16 4000 (256) 446 and 475.
template <typename S>
constexpr int64_t kLdsBlocks = sizeof(S) == 8 ? 256 : 512;
template <typename S, bool LDS>
struct SliceRows {
  int32_t row[LDS ? kSliceRows : 1];
  S r[LDS ? kSliceRows : 1];
  __device__ void load(const int32_t* __restrict__ rows, const S* __restrict__ res, bool by_row,
                       int s_begin, int cnt) {
    if constexpr (LDS) {
      const int t = threadIdx.x;
      if (t < cnt) {
        const int32_t i = rows[s_begin + t];
        row[t] = i;
        r[t] = res[by_row ? i : s_begin + t];
      }
      __syncthreads();
    }
  }
  // wave w takes rows w, w + kWaves, ... in order: get(row) then use(value, r)
  template <typename G, typename U>
  __device__ __forceinline__ void for_rows(const int32_t* __restrict__ rows,
                                           const S* __restrict__ res, bool by_row, int s_begin,
                                           int cnt, int wave, G&& get, U&& use) const {
    int s = wave;
    if constexpr (LDS) {
      for (; s + (kRowsAhead - 1) * kWaves < cnt; s += kRowsAhead * kWaves) {
        decltype(get(0)) b[kRowsAhead];
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) b[u] = get(row[s + u * kWaves]);
#pragma unroll
        for (int u = 0; u < kRowsAhead; ++u) use(b[u], r[s + u * kWaves]);
      }
      for (; s < cnt; s += kWaves) use(get(row[s]), r[s]);
    } else {
#pragma unroll 4
      for (; s < cnt; s += kWaves) {
        const int32_t i = rows[s_begin + s];
        use(get(i), res[by_row ? i : s_begin + s]);
      }
    }
  }
};

// part[slice][j] = sum over the slice's rows s of B[rows[s]][j] r[s].  A block
// covers 64*W columns (W per lane) and a slice of kSliceRows rows: wave w
// takes rows w, w+4, ... of the slice (so the four waves stream neighbouring
// rows), and the four wave sums are added in wave order through LDS.
template <typename S, bool VEC, bool LDS>
__global__ void __launch_bounds__(kBlock)
k_dense_colsum(int32_t n, int32_t nr, const int32_t* __restrict__ rows, const S* __restrict__ B,
               const S* __restrict__ r, bool by_row, S* __restrict__ part) {
  constexpr int W = VEC ? Vec<S>::N : 1;
  __shared__ S sh[kWaves][64 * W];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t c0 = (int64_t)blockIdx.x * 64 * W;
  const int64_t j0 = c0 + (int64_t)lane * W;
  const int slice = blockIdx.y;
  const int s0 = slice * kSliceRows, cnt = min(kSliceRows, nr - s0);
  __shared__ SliceRows<S, LDS> sl;
  sl.load(rows, r, by_row, s0, cnt);
  S acc[W];
#pragma unroll
  for (int w = 0; w < W; ++w) acc[w] = S(0);
  if (j0 < n) {
    if (VEC) {
      using V = typename Vec<S>::T;
      sl.for_rows(
          rows, r, by_row, s0, cnt, wave,
          [&](int32_t i) { return *reinterpret_cast<const V*>(B + (int64_t)i * n + j0); },
          [&](const V& b, S rs) {
            if constexpr (W == 4) {
              acc[0] += b.x * rs;
              acc[1] += b.y * rs;
              acc[2] += b.z * rs;
              acc[3] += b.w * rs;
            } else if constexpr (W == 2) {
              acc[0] += b.x * rs;
              acc[1] += b.y * rs;
            }
          });
    } else {
      sl.for_rows(
          rows, r, by_row, s0, cnt, wave, [&](int32_t i) { return B[(int64_t)i * n + j0]; },
          [&](S b, S rs) { acc[0] += b * rs; });
    }
  }
#pragma unroll
  for (int w = 0; w < W; ++w) sh[wave][lane * W + w] = acc[w];
  __syncthreads();
  // thread t adds column t of the block (and t + 256 when the block is wider)
  for (int c = threadIdx.x; c < 64 * W; c += kBlock) {
    if (c0 + c >= n) break;
    S v = sh[0][c];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += sh[w][c];
    part[(int64_t)slice * n + c0 + c] = v;
  }
}

// One block per 16 columns: lane group g = threadIdx.x / 16 (four per wave)
// adds slices g, g+16, ... of its column in FP64 (each group reads 64
// neighbouring bytes of a slice row), the 16 partial sums of a column are
// added in order of g through LDS, then Adagrad (or the fixed step) and the
// projection.
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_dense_update(int32_t n, int32_t n_slices, const S* __restrict__ part, S* __restrict__ q,
               S* __restrict__ A, StepArgs st) {
  constexpr int kCols = 16, kParts = kBlock / kCols;
  __shared__ double sh[kParts][kCols];
  const int c = threadIdx.x % kCols, g = threadIdx.x / kCols;
  const int64_t j = (int64_t)blockIdx.x * kCols + c;
  double gd = 0.0;
  if (j < n)
    for (int k = g; k < n_slices; k += kParts) gd += static_cast<double>(part[(int64_t)k * n + j]);
  sh[g][c] = gd;
  __syncthreads();
  if (threadIdx.x >= kCols || j >= n) return;
  gd = sh[0][c];
#pragma unroll
  for (int p = 1; p < kParts; ++p) gd += sh[p][c];
  const S g_j = static_cast<S>(gd);
  S v = q[j];
  if (st.optimizer == 0) {
    const S acc = A[j] + g_j * g_j;
    A[j] = acc;
    v -= static_cast<S>(st.eta) * g_j / (sqrt(acc) + static_cast<S>(st.eps));
  } else {
    v -= static_cast<S>(st.eta) * g_j;
  }
  q[j] = v > S(0) ? v : S(0);
}

// out[e] = sum over rows of r[e]^2 (FP64, fixed order: strided per thread, then a
// tree), one block per epoch.
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_dense_sq_sum(int32_t m, const S* __restrict__ r, double* __restrict__ out) {
  __shared__ double sh[kBlock];
  r += (int64_t)blockIdx.x * m;
  double s = 0.0;
  for (int i = threadIdx.x; i < m; i += kBlock) s += static_cast<double>(r[i]) * r[i];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = kBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = sh[0];
}

// ---- B stored as bf16 (FP32 arithmetic and state) -------------------------
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ float dot8(const uint4 b, const float4 q0, const float4 q1) {
  return bf16_lo(b.x) * q0.x + bf16_hi(b.x) * q0.y + bf16_lo(b.y) * q0.z + bf16_hi(b.y) * q0.w +
         bf16_lo(b.z) * q1.x + bf16_hi(b.z) * q1.y + bf16_lo(b.w) * q1.z + bf16_hi(b.w) * q1.w;
}

// r[s] = B[row] . q - y[row]; VEC: 16-byte rows (8 values per load)
template <bool VEC>
__global__ void __launch_bounds__(kBlock)
k_dense_resid_bf16(int32_t n, int32_t nr, const int32_t* __restrict__ rows,
                   const uint16_t* __restrict__ B, const float* __restrict__ y,
                   const float* __restrict__ q, float* __restrict__ r) {
  const int s = blockIdx.x * kWaves + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (s >= nr) return;
  const int32_t i = rows ? rows[s] : s;
  const uint16_t* row = B + (int64_t)i * n;
  float acc = 0.f;
  if (VEC) {
    const uint4* rv = reinterpret_cast<const uint4*>(row);
    const float4* qv = reinterpret_cast<const float4*>(q);
    const int nv = n / 8;
    float a2 = 0.f;
    int j = lane;
    for (; j + 64 < nv; j += 128) {   // two 16-byte loads in flight per lane
      const uint4 b0 = rv[j], b1 = rv[j + 64];
      acc += dot8(b0, qv[2 * j], qv[2 * j + 1]);
      a2 += dot8(b1, qv[2 * (j + 64)], qv[2 * (j + 64) + 1]);
    }
    if (j < nv) acc += dot8(rv[j], qv[2 * j], qv[2 * j + 1]);
    acc += a2;
  } else {
    for (int j = lane; j < n; j += 64) acc += __uint_as_float((uint32_t)row[j] << 16) * q[j];
  }
  acc = wave_sum(acc);
  if (lane == 0) r[s] = acc - y[i];
}

// part[slice][j] = sum over the slice's rows of B[rows[s]][j] r[s]; a lane
// covers 8 columns (one 16-byte load) in VEC mode, else 1.
template <bool VEC, bool LDS>
__global__ void __launch_bounds__(kBlock)
k_dense_colsum_bf16(int32_t n, int32_t nr, const int32_t* __restrict__ rows,
                    const uint16_t* __restrict__ B, const float* __restrict__ r, bool by_row,
                    float* __restrict__ part) {
  constexpr int W = VEC ? 8 : 1;
  __shared__ float sh[kWaves][64 * W];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t c0 = (int64_t)blockIdx.x * 64 * W;
  const int64_t j0 = c0 + (int64_t)lane * W;
  const int slice = blockIdx.y;
  const int s0 = slice * kSliceRows, cnt = min(kSliceRows, nr - s0);
  __shared__ SliceRows<float, LDS> sl;
  sl.load(rows, r, by_row, s0, cnt);
  float acc[W];
#pragma unroll
  for (int w = 0; w < W; ++w) acc[w] = 0.f;
  if (j0 < n) {
    if (VEC)
      sl.for_rows(
          rows, r, by_row, s0, cnt, wave,
          [&](int32_t i) { return *reinterpret_cast<const uint4*>(B + (int64_t)i * n + j0); },
          [&](const uint4& b, float rs) {
            acc[0] += bf16_lo(b.x) * rs;
            acc[1] += bf16_hi(b.x) * rs;
            acc[2] += bf16_lo(b.y) * rs;
            acc[3] += bf16_hi(b.y) * rs;
            acc[4] += bf16_lo(b.z) * rs;
            acc[5] += bf16_hi(b.z) * rs;
            acc[6] += bf16_lo(b.w) * rs;
            acc[7] += bf16_hi(b.w) * rs;
          });
    else
      sl.for_rows(
          rows, r, by_row, s0, cnt, wave, [&](int32_t i) { return B[(int64_t)i * n + j0]; },
          [&](uint16_t b, float rs) { acc[0] += __uint_as_float((uint32_t)b << 16) * rs; });
  }
#pragma unroll
  for (int w = 0; w < W; ++w) sh[wave][lane * W + w] = acc[w];
  __syncthreads();
  for (int c = threadIdx.x; c < 64 * W; c += kBlock) {
    if (c0 + c >= n) break;
    float v = sh[0][c];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += sh[w][c];
    part[(int64_t)slice * n + c0 + c] = v;
  }
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// Epochs of minibatches: residual, column sums, update.  With a loss history
// the residuals of all rows follow each epoch, in natural order (res[e]); an
// epoch whose first minibatch holds every row takes its residuals from there
// (the same rows, the same q), and the squares are summed once per block of
// epochs.
template <typename S, typename R, typename C>
hipError_t epochs(const DenseArgs& a, int cols_per_block, R&& resid, C&& colsum, hipStream_t s) {
  S* q = static_cast<S*>(a.q);
  S* A = static_cast<S*>(a.A);
  S* part = static_cast<S*>(a.part);
  const unsigned col_blocks = blocks_for(a.n, cols_per_block);
  const bool whole = a.chunk >= a.m;
  const S* last = nullptr;   // residuals of all rows at the current q
  for (int32_t e = 0; e < a.E; ++e) {
    for (int32_t s0 = 0; s0 < a.m; s0 += a.chunk) {
      const int32_t nr = std::min(a.chunk, a.m - s0);
      const int32_t* rows = a.perms + (int64_t)e * a.m + s0;
      const int32_t n_slices = (nr + kSliceRows - 1) / kSliceRows;
      const bool kept = whole && last;
      S* r = static_cast<S*>(a.r);
      if (!kept) resid(dim3(blocks_for(nr, kWaves)), nr, rows, r);
      colsum(dim3(col_blocks, n_slices), nr, rows, kept ? last : r, kept, part);
      hipLaunchKernelGGL(k_dense_update<S>, dim3(blocks_for(a.n, 16)), dim3(kBlock), 0, s, a.n,
                         n_slices, part, q, A, a.st);
    }
    if (a.loss) {
      const int32_t k = e % a.loss_epochs;
      S* all = static_cast<S*>(a.res) + (int64_t)k * a.m;
      resid(dim3(blocks_for(a.m, kWaves)), a.m, (const int32_t*)nullptr, all);
      last = all;
      if (k == a.loss_epochs - 1 || e == a.E - 1)
        hipLaunchKernelGGL(k_dense_sq_sum<S>, dim3(k + 1), dim3(kBlock), 0, s, a.m,
                           static_cast<const S*>(a.res), a.loss + (e - k));
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

template <typename S, bool VEC>
hipError_t run(const DenseArgs& a, hipStream_t s) {
  const S* B = static_cast<const S*>(a.B);
  const S* y = static_cast<const S*>(a.y);
  const S* q = static_cast<const S*>(a.q);
  return epochs<S>(
      a, 64 * (VEC ? Vec<S>::N : 1),
      [&](dim3 grid, int32_t nr, const int32_t* rows, S* r) {
        hipLaunchKernelGGL((k_dense_resid<S, VEC>), grid, dim3(kBlock), 0, s, a.n, nr, rows, B, y, q,
                           r);
      },
      [&](dim3 grid, int32_t nr, const int32_t* rows, const S* r, bool by_row, S* part) {
        auto go = [&](auto kern) {
          hipLaunchKernelGGL(kern, grid, dim3(kBlock), 0, s, a.n, nr, rows, B, r, by_row, part);
        };
        if ((int64_t)grid.x * grid.y <= kLdsBlocks<S>)
          go(k_dense_colsum<S, VEC, true>);
        else
          go(k_dense_colsum<S, VEC, false>);
      },
      s);
}

template <bool VEC>
hipError_t run_bf16(const DenseArgs& a, hipStream_t s) {
  const uint16_t* B = static_cast<const uint16_t*>(a.B);
  const float* y = static_cast<const float*>(a.y);
  const float* q = static_cast<const float*>(a.q);
  return epochs<float>(
      a, 64 * (VEC ? 8 : 1),
      [&](dim3 grid, int32_t nr, const int32_t* rows, float* r) {
        hipLaunchKernelGGL(k_dense_resid_bf16<VEC>, grid, dim3(kBlock), 0, s, a.n, nr, rows, B, y, q,
                           r);
      },
      [&](dim3 grid, int32_t nr, const int32_t* rows, const float* r, bool by_row, float* part) {
        auto go = [&](auto kern) {
          hipLaunchKernelGGL(kern, grid, dim3(kBlock), 0, s, a.n, nr, rows, B, r, by_row, part);
        };
        if ((int64_t)grid.x * grid.y <= kLdsBlocks<float>)
          go(k_dense_colsum_bf16<VEC, true>);
        else
          go(k_dense_colsum_bf16<VEC, false>);
      },
      s);
}

}  // namespace

int32_t dense_slice_rows() { return kSliceRows; }

hipError_t dense_spgd_bf16(const DenseArgs& a, bool vec, hipStream_t s) {
  return vec ? run_bf16<true>(a, s) : run_bf16<false>(a, s);
}

hipError_t dense_spgd(const DenseArgs& a, bool f64, bool vec, hipStream_t s) {
  if (f64) return vec ? run<double, true>(a, s) : run<double, false>(a, s);
  return vec ? run<float, true>(a, s) : run<float, false>(a, s);
}
