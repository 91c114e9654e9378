// Dynamic assignment ratios from link speeds (section "Dynamic assignment
// ratio", eqs. "dar2"/"dar" and Example "DAR matrix computation"; section
// "Link/path travel time", eq. "cost").
//
// Time is in minutes and observation intervals are [h*dt, (h+1)*dt).  A link
// entered at time t is crossed in len/speed(interval of t); the last
// interval's speed holds after the end of the day.  A vehicle of path k
// departing at t enters the path's i-th link at tau_i(t): tau_0(t) = t,
// tau_{i+1}(t) = tau_i(t) + c(tau_i(t)).  Departure interval h maps onto the
// arrival window [tau_i(h dt), tau_i((h+1) dt)] at that link, and the ratio of
// observation interval h2 is the share of the window inside it.
//
// Paths of up to 16 segments of links take one kernel (k_ratios below); longer
// ones two kernels per chunk of days:
//   k_trajectories  one thread per (eight days, path, boundary b in 0..H): the travel
//                   time from the b*dt departure to the entry of every link of
//                   the path, traj[day][pair][b] (pairs = (path, i) in path
//                   order), and optionally the whole path's travel time (the
//                   path cost of eq. "cost" for a departure at b*dt), whose
//                   day mean k_exit_sums forms;
//   k_dar_windows   one thread per (pair, departure interval h): the shares
//                   of the day windows, [r_h, dt + r_{h+1}] relative to h*dt,
//                   summed over the chunk's days in order, added into the
//                   running sums; the last chunk divides by the day count.
//                   The share of interval h+l is F((l+1) dt) - F(l dt), with
//                   F(x) = clamp((x - lo) / w, 0, 1) the fraction of the window
//                   before x (the window's overlap with the interval over w).
// Keeping times relative to the departure keeps the window arithmetic at the
// precision of travel times (tens of minutes), not of times of day.
//
// Mean path travel times (eqs. "cost", "logit", "rt"): the same walk from the
// departure at t*dt to the exit of the path's last link, for every day of a
// pattern, averaged over the days.  Two kernels:
//   k_path_cost_slices  one thread per (slice of days, path, t), t fastest:
//                       the FP64 sum of the slice's day costs; four days walk
//                       the path together (the link index and length are
//                       loaded once, four speed loads are in flight);
//   k_cost_mean         one thread per (path, t): the slice sums in slice
//                       order, divided by the day count.
#include "dode_internal.h"

#include <algorithm>

namespace {

constexpr int kBlock = 256;
constexpr int kTrajDays = 8;   // days walked together by one trajectory thread

template <typename S>
__device__ __forceinline__ S link_time(const S* __restrict__ len, const S* __restrict__ speed_day,
                                       int32_t H_speed, S dt, int32_t a, S t) {
  int64_t h = static_cast<int64_t>(floor(t / dt));
  h = h < 0 ? 0 : (h >= H_speed ? H_speed - 1 : h);
  return len[a] / speed_day[(int64_t)a * H_speed + h];
}

// One thread per (group of eight days, path, boundary b), b fastest: the
// eight days' trajectories are walked together, so eight independent chains
// of speed gathers are in flight (days past the chunk repeat its last day and
// are not stored).
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_trajectories(int32_t n_paths, const int32_t* __restrict__ path_ptr,
               const int32_t* __restrict__ path_link, int32_t L, const S* __restrict__ len,
               const S* __restrict__ speed, int32_t day0, int32_t n_days, int32_t H_speed, S dt,
               int32_t H, int64_t n_pairs, S* __restrict__ traj, S* __restrict__ exit_time) {
  // The entry time t0 + r is a sum of its own, never fused with the product
  // b * dt: which interval's speed a link takes is decided by the rounded sum.
#pragma clang fp contract(off)
  constexpr int kDays = kTrajDays;
  const int64_t per_group = (int64_t)n_paths * (H + 1);
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int32_t n_groups = (n_days + kDays - 1) / kDays;
  if (idx >= per_group * n_groups) return;
  const int32_t dg = (int32_t)(idx / per_group);
  const int64_t kb = idx % per_group;   // k * (H+1) + b
  const int32_t k = (int32_t)(kb / (H + 1));
  const int32_t b = (int32_t)(kb % (H + 1));
  const int64_t day_stride = (int64_t)L * H_speed, traj_stride = n_pairs * (H + 1);
  const S* sp[kDays];
  S* out[kDays];
  bool on[kDays];
#pragma unroll
  for (int u = 0; u < kDays; ++u) {
    const int32_t d = min(dg * kDays + u, n_days - 1);
    on[u] = dg * kDays + u < n_days;
    sp[u] = speed + (int64_t)(day0 + d) * day_stride;
    out[u] = traj + (int64_t)d * traj_stride;
  }
  const S t0 = static_cast<S>(b) * dt;
  S r[kDays];   // travel time so far
#pragma unroll
  for (int u = 0; u < kDays; ++u) r[u] = S(0);
  for (int32_t m = path_ptr[k]; m < path_ptr[k + 1]; ++m) {
    const int32_t a = path_link[m];
#pragma unroll
    for (int u = 0; u < kDays; ++u) {
      if (on[u]) out[u][(int64_t)m * (H + 1) + b] = r[u];
      r[u] += link_time(len, sp[u], H_speed, dt, a, t0 + r[u]);
    }
  }
  if (exit_time)   // [d][k][b]: the whole path's travel time
#pragma unroll
    for (int u = 0; u < kDays; ++u)
      if (on[u]) exit_time[(int64_t)(dg * kDays + u) * per_group + kb] = r[u];
}

// Running FP64 sums of the chunk's path travel times, days in order, for the
// departures at the interval starts (boundaries b < H); the last chunk writes
// cost[t][k] = sum / n_days.
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_exit_sums(int32_t n_paths, int32_t H, int32_t n_days_chunk, const S* __restrict__ exit_time,
            bool first_chunk, bool last_chunk, int32_t n_days_total, double* __restrict__ sums,
            S* __restrict__ cost) {
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= (int64_t)n_paths * H) return;
  const int32_t k = (int32_t)(idx / H), t = (int32_t)(idx % H);
  const int64_t per_day = (int64_t)n_paths * (H + 1);
  const S* e = exit_time + (int64_t)k * (H + 1) + t;
  double s = first_chunk ? 0.0 : sums[idx];
  for (int32_t d = 0; d < n_days_chunk; ++d) s += static_cast<double>(e[d * per_day]);
  if (last_chunk)
    cost[(int64_t)t * n_paths + k] = static_cast<S>(s / n_days_total);
  else
    sums[idx] = s;
}

// 1 / w for the window shares: the hardware reciprocal in FP32 (within 1 ulp;
// the kernel is bound by its instruction count), the quotient in FP64.
__device__ __forceinline__ float share_recip(float w) { return __builtin_amdgcn_rcpf(w); }
__device__ __forceinline__ double share_recip(double w) { return 1.0 / w; }
// min(max(x, 0), 1): one v_med3 in FP32
__device__ __forceinline__ float clamp01(float x) { return __builtin_amdgcn_fmed3f(x, 0.f, 1.f); }
__device__ __forceinline__ double clamp01(double x) { return x < 0.0 ? 0.0 : (x > 1.0 ? 1.0 : x); }

template <typename S, int KMAX>
__global__ void __launch_bounds__(kBlock)
k_dar_windows(int64_t n_pairs, int32_t n_days_chunk, int32_t H, int32_t K, S dt,
              const S* __restrict__ traj, bool first_chunk, bool last_chunk, int32_t n_days_total,
              S* __restrict__ Rr) {
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= n_pairs * H) return;
  const int64_t m = idx / H;
  const int32_t h = (int32_t)(idx % H);
  const int kk = min(K, H - h);   // lags that stay inside the day
  S acc[KMAX];
#pragma unroll
  for (int l = 0; l < KMAX; ++l) acc[l] = first_chunk || l >= K ? S(0) : Rr[((int64_t)l * H + h) * n_pairs + m];
  const int64_t day_stride = n_pairs * (H + 1);
  const S* tr = traj + m * (H + 1) + h;
  // interval h+l ends at (l+1)*dt relative to the departure
  S edge[KMAX];
#pragma unroll
  for (int l = 0; l < KMAX; ++l) edge[l] = static_cast<S>(l + 1) * dt;
  // One day's window [lo, hi] (relative to h*dt; observation interval h+l is
  // [l*dt, (l+1)*dt)) added into acc.  Every lag is accumulated; lags past the
  // day (l >= kk) are written as zeros below.
  auto add_day = [&](S lo, S hi) {
    // FIFO violation (hi < lo): the window between the two end points
    const S a0 = fmin(lo, hi), w = fmax(lo, hi) - a0;
    if (w <= S(0)) {   // all of the interval arrives at one instant
      const int la = static_cast<int>(fmin(floor(a0 / dt), static_cast<S>(KMAX)));
#pragma unroll
      for (int ll = 0; ll < KMAX; ++ll)
        if (ll == la) acc[ll] += S(1);
      return;
    }
    const S inv_w = share_recip(w);
    S f_prev = S(0);   // F(0) = 0: windows start at or after their departure
#pragma unroll
    for (int ll = 0; ll < KMAX; ++ll) {
      const S f = clamp01((edge[ll] - a0) * inv_w);
      acc[ll] += f - f_prev;
      f_prev = f;
    }
  };
  // days in order: groups of eight whose loads are in flight together, then
  // the rest one by one
  constexpr int kDays = 8;
  const S* p = tr;
  int32_t d = 0;
  for (; d + kDays <= n_days_chunk; d += kDays, p += kDays * day_stride) {
    S lo[kDays], hi[kDays];
#pragma unroll
    for (int u = 0; u < kDays; ++u) {
      lo[u] = p[u * day_stride];
      hi[u] = dt + p[u * day_stride + 1];
    }
#pragma unroll
    for (int u = 0; u < kDays; ++u) add_day(lo[u], hi[u]);
  }
  for (; d < n_days_chunk; ++d, p += day_stride) add_day(p[0], dt + p[1]);
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    if (l >= K) break;
    const S v = l >= kk ? S(0) : (last_chunk ? acc[l] / static_cast<S>(n_days_total) : acc[l]);
    Rr[((int64_t)l * H + h) * n_pairs + m] = v;
  }
}

// The whole ratio construction of several patterns in one kernel: no
// trajectory leaves the chip.
//
// A block owns one path and 63 departure intervals of one pattern: lane i
// walks the boundary departure b0 + i, and the window of interval b0 + i needs
// its own and the next lane's entry times (lane 63 only supplies lane 62).  The
// path's links are cut into segments of SEG, one per wave, whose shares stay in
// registers (SEG x KMAX sums per lane) over all days; wave s takes the travel
// times of ND days from wave s-1 through LDS and passes them on, so the waves
// form a pipeline over the groups of days, one step per barrier.  The speed
// gathers of a link are in flight while its windows are added.  Days are added
// in order, so the results are those of the two kernels above for any grouping.
// Where a pattern's blocks are too few to fill the chip (dar_split), its days are
// split over parts (blockIdx.y), whose sums k_join_parts adds in order.
//
// What bounds it: the VALU (about 45 instructions per day, link and boundary
// in FP32) and the chain of gathers along a path.  The trajectories of the two
// kernels above (4 bytes per day, link and boundary, written, read twice, and a
// scratch allocation of up to 4 GiB that the call's own synchronisation
// gives back each time) took 52 ms for 365 days of 450 paths of 20 links at
// 288 intervals and 6 lags in 4 patterns, of which 3.6 ms were kernels.
constexpr int kMaxSegs = 16;   // waves of a block
constexpr int kPatterns = 16;  // patterns of one launch
struct PatternDays {
  int32_t ptr[kPatterns + 1];
  int32_t parts[kPatterns];
};

// RN(t / dt) with rdt = RN(1 / dt): two residual steps on the approximate
// quotient, the second of which rounds correctly (Markstein, IBM J. Res. Dev.
// 34, 1990).  The interval of an entry time is decided by this quotient.
__device__ __forceinline__ float quotient(float t, float dt, float rdt) {
  float q = t * rdt;
  q = __builtin_fmaf(__builtin_fmaf(-q, dt, t), rdt, q);
  return __builtin_fmaf(__builtin_fmaf(-q, dt, t), rdt, q);
}
__device__ __forceinline__ double quotient(double t, double dt, double) { return t / dt; }

// value of the next lane (lane 63 keeps its own)
__device__ __forceinline__ float next_lane(float x) { return __shfl_down(x, 1, 64); }
__device__ __forceinline__ double next_lane(double x) { return __shfl_down(x, 1, 64); }

template <typename S, int KMAX, int SEG, int ND>
__global__ void __launch_bounds__(64 * kMaxSegs)
k_ratios(int32_t n_paths, const int32_t* __restrict__ path_ptr,
         const int32_t* __restrict__ path_link, int32_t L, const S* __restrict__ len,
         const S* __restrict__ speed, PatternDays days, int32_t H_speed, S dt, S rdt, int32_t H,
         int32_t K, int64_t n_pairs, S* __restrict__ Rr, S* __restrict__ cost,
         double* __restrict__ part_exit, S* __restrict__ part_sum) {
#pragma clang fp contract(off)   // as in k_trajectories
  constexpr int kWin = 63;
  extern __shared__ __align__(16) unsigned char hand_mem[];
  S* hand = reinterpret_cast<S*>(hand_mem);   // [2][waves][ND][64]
  const int nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n_chunks = (H + kWin - 1) / kWin;
  int item = blockIdx.x;
  const int chunk = item % n_chunks;
  item /= n_chunks;
  const int k = item % n_paths, q = item / n_paths;
  // the block's days: whole groups, a part of the pattern's
  const int all = days.ptr[q + 1] - days.ptr[q], n_parts = days.parts[q];
  if ((int)blockIdx.y >= n_parts) return;
  const int per = ((all + ND - 1) / ND + n_parts - 1) / n_parts * ND;
  const int skip = min(all, (int)blockIdx.y * per);
  const int d_begin = days.ptr[q] + skip, n_days = min(per, all - skip);
  const int m0 = path_ptr[k], m_end = path_ptr[k + 1];
  const int n_segs = max(1, (m_end - m0 + SEG - 1) / SEG);
  const int m = m0 + wave * SEG;   // first pair of the wave's segment
  const int n_links = wave < n_segs ? min(SEG, m_end - m) : 0;
  const int b = min(chunk * kWin + lane, H);
  const S t0 = static_cast<S>(b) * dt;
  const int64_t day_stride = (int64_t)L * H_speed;
  // the segment's links (uniform)
  int64_t row[SEG];
  S ln[SEG];
#pragma unroll
  for (int i = 0; i < SEG; ++i)
    if (i < n_links) {
      const int a = path_link[m + i];
      row[i] = (int64_t)a * H_speed;
      ln[i] = len[a];
    }
  S edge[KMAX], acc[SEG][KMAX];
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    edge[l] = static_cast<S>(l + 1) * dt;
#pragma unroll
    for (int i = 0; i < SEG; ++i) acc[i][l] = S(0);
  }
  double exit_sum = 0.0;
  const int n_groups = (n_days + ND - 1) / ND;
  const S h_last = static_cast<S>(H_speed - 1);
  for (int st = 0; st < n_groups + n_segs - 1; ++st) {
    const int g = st - wave;
    if (wave < n_segs && g >= 0 && g < n_groups) {
      const int d0 = g * ND, nd = min(ND, n_days - d0);
      const S* sp = speed + (int64_t)(d_begin + d0) * day_stride;
      S r[ND];
#pragma unroll
      for (int u = 0; u < ND; ++u)
        r[u] = wave == 0 ? S(0)
                         : hand[((((st + 1) & 1) * nw + wave - 1) * ND + u) * 64 + lane];
#pragma unroll
      for (int i = 0; i < SEG; ++i) {
        if (i < n_links) {
          // entry intervals and speeds (days past the pattern repeat its last)
          S v[ND];
#pragma unroll
          for (int u = 0; u < ND; ++u) {
            const S f = floor(quotient(t0 + r[u], dt, rdt));
            const int h = static_cast<int>(fmax(fmin(f, h_last), S(0)));
            v[u] = (sp + (int64_t)min(u, nd - 1) * day_stride + row[i])[(uint32_t)h];
          }
          // the link's window shares (as in k_dar_windows)
#pragma unroll
          for (int u = 0; u < ND; ++u) {
            if (u < nd) {
              const S lo = r[u], hi = dt + next_lane(r[u]);
              const S a0 = fmin(lo, hi), w = fmax(lo, hi) - a0;
              if (w <= S(0)) {
                const int la = static_cast<int>(fmin(floor(a0 / dt), static_cast<S>(KMAX)));
#pragma unroll
                for (int l = 0; l < KMAX; ++l)
                  if (l == la) acc[i][l] += S(1);
              } else {
                const S inv_w = share_recip(w);
                S f_prev = S(0);
#pragma unroll
                for (int l = 0; l < KMAX; ++l) {
                  const S f = clamp01((edge[l] - a0) * inv_w);
                  acc[i][l] += f - f_prev;
                  f_prev = f;
                }
              }
            }
          }
#pragma unroll
          for (int u = 0; u < ND; ++u) r[u] += ln[i] / v[u];
        }
      }
      if (wave == n_segs - 1) {
#pragma unroll
        for (int u = 0; u < ND; ++u)
          if (u < nd) exit_sum += static_cast<double>(r[u]);
      } else {
#pragma unroll
        for (int u = 0; u < ND; ++u)
          hand[(((st & 1) * nw + wave) * ND + u) * 64 + lane] = r[u];
      }
    }
    __syncthreads();
  }
  const int h = chunk * kWin + lane;   // the lane's interval
  if (lane == kWin || h >= H) return;
  if (n_parts > 1) {
    const int64_t row = (int64_t)blockIdx.y * (gridDim.x / (n_paths * n_chunks)) + q;
    if (wave == n_segs - 1) part_exit[(row * H + h) * n_paths + k] = exit_sum;
#pragma unroll
    for (int l = 0; l < KMAX; ++l)
      if (l < K) {
        S* out = part_sum + ((row * K + l) * H + h) * n_pairs + m;
#pragma unroll
        for (int i = 0; i < SEG; ++i)
          if (i < n_links) out[i] = acc[i][l];
      }
    return;
  }
  if (cost && wave == n_segs - 1)
    cost[((int64_t)q * H + h) * n_paths + k] = static_cast<S>(exit_sum / n_days);
  const int kk = min(K, H - h);   // lags that stay inside the day
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    if (l < K) {
      S* out = Rr + (((int64_t)q * K + l) * H + h) * n_pairs + m;
#pragma unroll
      for (int i = 0; i < SEG; ++i)
        if (i < n_links) out[i] = l >= kk ? S(0) : acc[i][l] / static_cast<S>(n_days);
    }
  }
}

// Means over the days of pattern blockIdx.y from the sums of its parts, if it has
// several: ratios (idx below K*H*n_pairs), then path costs.
template <typename S>
__global__ void __launch_bounds__(kBlock)
k_join_parts(PatternDays days, int32_t n_paths, int64_t n_pairs, int32_t H, int32_t K,
             const double* __restrict__ part_exit, const S* __restrict__ part_sum,
             S* __restrict__ Rr, S* __restrict__ cost) {
  const int q = blockIdx.y, nq = gridDim.y, n_days = days.ptr[q + 1] - days.ptr[q];
  const int n_parts = days.parts[q];
  if (n_parts == 1) return;
  const int64_t n_r = (int64_t)K * H * n_pairs, n_c = (int64_t)H * n_paths;
  int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n_r) {
    const int l = (int)(i / (H * n_pairs)), h = (int)(i / n_pairs % H);
    S s = S(0);
    for (int p = 0; p < n_parts; ++p) s += part_sum[((int64_t)p * nq + q) * n_r + i];
    Rr[q * n_r + i] = l >= min(K, H - h) ? S(0) : s / static_cast<S>(n_days);
    return;
  }
  i -= n_r;
  if (!cost || i >= n_c) return;
  double s = 0.0;
  for (int p = 0; p < n_parts; ++p) s += part_exit[((int64_t)p * nq + q) * n_c + i];
  cost[q * n_c + i] = static_cast<S>(s / n_days);
}

template <typename S>
__global__ void __launch_bounds__(kBlock)
k_path_cost_slices(int32_t n_paths, const int32_t* __restrict__ path_ptr,
                   const int32_t* __restrict__ path_link, int32_t L, const S* __restrict__ len,
                   const S* __restrict__ speed, int32_t n_days, int32_t per_slice, int32_t n_slices,
                   int32_t H_speed, S dt, int32_t T, double* __restrict__ partial) {
#pragma clang fp contract(off)   // as in k_trajectories
  const int64_t per = (int64_t)n_paths * T;
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= per * n_slices) return;
  const int32_t g = (int32_t)(idx / per);
  const int32_t k = (int32_t)((idx % per) / T);
  const int32_t t = (int32_t)(idx % T);
  const S t0 = static_cast<S>(t) * dt;
  const int32_t m0 = path_ptr[k], m1 = path_ptr[k + 1];
  const int32_t d_begin = g * per_slice, d_end = min(n_days, d_begin + per_slice);
  constexpr int kDays = 4;
  const int64_t day_stride = (int64_t)L * H_speed;
  double sum = 0.0;
  for (int32_t d0 = d_begin; d0 < d_end; d0 += kDays) {
    const S* sp[kDays];
    S r[kDays];
#pragma unroll
    for (int u = 0; u < kDays; ++u) {
      sp[u] = speed + (int64_t)min(d0 + u, d_end - 1) * day_stride;
      r[u] = S(0);
    }
    for (int32_t m = m0; m < m1; ++m) {
      const int32_t a = path_link[m];
#pragma unroll
      for (int u = 0; u < kDays; ++u) r[u] += link_time(len, sp[u], H_speed, dt, a, t0 + r[u]);
    }
#pragma unroll
    for (int u = 0; u < kDays; ++u)
      if (d0 + u < d_end) sum += static_cast<double>(r[u]);
  }
  partial[idx] = sum;
}

template <typename S>
__global__ void __launch_bounds__(kBlock)
k_cost_mean(int32_t n_paths, int32_t T, int32_t n_slices, int32_t n_days,
            const double* __restrict__ partial, S* __restrict__ cost) {
  const int64_t per = (int64_t)n_paths * T;
  const int64_t idx = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (idx >= per) return;
  const int32_t k = (int32_t)(idx / T), t = (int32_t)(idx % T);
  double s = 0.0;
  for (int32_t g = 0; g < n_slices; ++g) s += partial[g * per + idx];
  cost[(int64_t)t * n_paths + k] = static_cast<S>(s / n_days);
}

template <typename S>
__global__ void k_check_speeds(const S* __restrict__ x, int64_t n, int32_t* __restrict__ flag) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    if (!(x[i] > S(0)) || !isfinite(x[i])) *flag = 1;
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

template <typename S>
hipError_t run(int32_t n_paths, const int32_t* path_ptr, const int32_t* path_link, int64_t n_pairs,
               int32_t L, const S* len, const S* speed, int32_t n_days, int32_t H_speed, S dt,
               int32_t H, int32_t K, S* traj, int32_t chunk, S* Rr, S* exit_time, double* sums,
               S* cost, hipStream_t s) {
  for (int32_t d0 = 0; d0 < n_days; d0 += chunk) {
    const int32_t nd = std::min(chunk, n_days - d0);
    const int64_t n1 = (int64_t)((nd + kTrajDays - 1) / kTrajDays) * n_paths * (H + 1);
    hipLaunchKernelGGL(k_trajectories<S>, dim3(blocks_for(n1)), dim3(kBlock), 0, s, n_paths,
                       path_ptr, path_link, L, len, speed, d0, nd, H_speed, dt, H, n_pairs, traj,
                       cost ? exit_time : nullptr);
    const bool first = d0 == 0, last = d0 + nd >= n_days;
    if (cost)
      hipLaunchKernelGGL(k_exit_sums<S>, dim3(blocks_for((int64_t)n_paths * H)), dim3(kBlock), 0, s,
                         n_paths, H, nd, exit_time, first, last, n_days, sums, cost);
    // the window loop is unrolled to KMAX lags: the common K = 6 gets its own
    if (K <= 6)
      hipLaunchKernelGGL((k_dar_windows<S, 6>), dim3(blocks_for(n_pairs * H)), dim3(kBlock), 0, s,
                         n_pairs, nd, H, K, dt, traj, first, last, n_days, Rr);
    else if (K <= 8)
      hipLaunchKernelGGL((k_dar_windows<S, 8>), dim3(blocks_for(n_pairs * H)), dim3(kBlock), 0, s,
                         n_pairs, nd, H, K, dt, traj, first, last, n_days, Rr);
    else
      hipLaunchKernelGGL((k_dar_windows<S, kMaxDarLags>), dim3(blocks_for(n_pairs * H)),
                         dim3(kBlock), 0, s, n_pairs, nd, H, K, dt, traj, first, last, n_days, Rr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Links per wave and days in flight of the fused kernel: the sums of a segment
// take SEG * KMAX registers (two each in FP64).
template <typename S, int KMAX>
struct Seg {
  static constexpr int kLinks = sizeof(S) == 4 ? (KMAX <= 8 ? 8 : 4) : (KMAX <= 8 ? 4 : 2);
  static constexpr int kDays = sizeof(S) == 4 ? 8 : (KMAX <= 8 ? 4 : 2);
};

template <typename S, int KMAX>
hipError_t run_fused(int32_t n_paths, const int32_t* path_ptr, const int32_t* path_link,
                     int64_t n_pairs, int32_t longest, int32_t L, const S* len, const S* speed,
                     int32_t n_patterns, const int32_t* pattern_ptr, int32_t H_speed, S dt,
                     int32_t H, int32_t K, S* Rr, S* cost, const DarSplit& split, void* scratch,
                     hipStream_t s) {
  constexpr int SEG = Seg<S, KMAX>::kLinks, ND = Seg<S, KMAX>::kDays;
  const int nw = std::max(1, (longest + SEG - 1) / SEG);
  const int64_t per = (int64_t)n_paths * ((H + 62) / 63);
  const size_t lds = (size_t)2 * nw * ND * 64 * sizeof(S);
  if (split.per_launch < 1) return hipErrorInvalidValue;
  for (int32_t q0 = 0; q0 < n_patterns; q0 += split.per_launch) {
    const int32_t nq = std::min(split.per_launch, n_patterns - q0);
    PatternDays pd{};
    int32_t most = 1;   // parts of a pattern
    pd.ptr[0] = pattern_ptr[q0];
    for (int32_t q = 0; q < nq; ++q) {
      pd.ptr[q + 1] = pattern_ptr[q0 + q + 1];
      most = std::max(most, pd.parts[q] = split.parts[q0 + q]);
    }
    double* exits = static_cast<double*>(scratch);
    S* sums = reinterpret_cast<S*>(exits + (int64_t)most * nq * H * n_paths);
    S* rq = Rr + (int64_t)q0 * K * H * n_pairs;
    S* cq = cost ? cost + (int64_t)q0 * H * n_paths : nullptr;
    hipLaunchKernelGGL((k_ratios<S, KMAX, SEG, ND>), dim3((unsigned)(per * nq), most), dim3(64 * nw),
                       lds, s, n_paths, path_ptr, path_link, L, len, speed, pd, H_speed, dt,
                       static_cast<S>(1) / dt, H, K, n_pairs, rq, cq, exits, sums);
    if (most > 1)
      hipLaunchKernelGGL(k_join_parts<S>,
                         dim3(blocks_for((int64_t)K * H * n_pairs + (int64_t)H * n_paths), nq),
                         dim3(kBlock), 0, s, pd, n_paths, n_pairs, H, K, exits, sums, rq, cq);
  }
  return hipGetLastError();
}

template <typename S>
hipError_t fused(int32_t n_paths, const int32_t* path_ptr, const int32_t* path_link,
                 int64_t n_pairs, int32_t longest, int32_t L, const void* len, const void* speed,
                 int32_t n_patterns, const int32_t* pattern_ptr, int32_t H_speed, double dt,
                 int32_t H, int32_t K, void* Rr, void* cost, const DarSplit& split, void* scratch,
                 hipStream_t s) {
  auto go = [&](auto kmax) {
    return run_fused<S, decltype(kmax)::value>(
        n_paths, path_ptr, path_link, n_pairs, longest, L, static_cast<const S*>(len),
        static_cast<const S*>(speed), n_patterns, pattern_ptr, H_speed, static_cast<S>(dt), H, K,
        static_cast<S*>(Rr), static_cast<S*>(cost), split, scratch, s);
  };
  if (K <= 3) return go(std::integral_constant<int, 3>{});
  if (K <= 6) return go(std::integral_constant<int, 6>{});
  if (K <= 8) return go(std::integral_constant<int, 8>{});
  return go(std::integral_constant<int, kMaxDarLags>{});
}

template <typename S>
hipError_t run_costs(int32_t n_paths, const int32_t* path_ptr, const int32_t* path_link, int32_t L,
                     const S* len, const S* speed, int32_t n_days, int32_t H_speed, S dt, int32_t T,
                     int32_t per_slice, double* partial, S* cost, hipStream_t s) {
  const int32_t n_slices = (n_days + per_slice - 1) / per_slice;
  const int64_t per = (int64_t)n_paths * T;
  hipLaunchKernelGGL(k_path_cost_slices<S>, dim3(blocks_for(per * n_slices)), dim3(kBlock), 0, s,
                     n_paths, path_ptr, path_link, L, len, speed, n_days, per_slice, n_slices,
                     H_speed, dt, T, partial);
  hipLaunchKernelGGL(k_cost_mean<S>, dim3(blocks_for(per)), dim3(kBlock), 0, s, n_paths, T,
                     n_slices, n_days, partial, cost);
  return hipGetLastError();
}

}  // namespace

hipError_t path_costs(bool f64, int32_t n_paths, const int32_t* path_ptr, const int32_t* path_link,
                      int32_t L, const void* len, const void* speed, int32_t n_days, int32_t H_speed,
                      double dt, int32_t T, int32_t per_slice, double* partial, void* cost,
                      hipStream_t s) {
  if (f64)
    return run_costs<double>(n_paths, path_ptr, path_link, L, static_cast<const double*>(len),
                             static_cast<const double*>(speed), n_days, H_speed, dt, T, per_slice,
                             partial, static_cast<double*>(cost), s);
  return run_costs<float>(n_paths, path_ptr, path_link, L, static_cast<const float*>(len),
                          static_cast<const float*>(speed), n_days, H_speed, static_cast<float>(dt),
                          T, per_slice, partial, static_cast<float*>(cost), s);
}

hipError_t dar_check_speeds(bool f64, const void* speed, int64_t n, int32_t* flag, hipStream_t s) {
  const unsigned b = (unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, blocks_for(n)));
  if (f64)
    hipLaunchKernelGGL(k_check_speeds<double>, dim3(b), dim3(kBlock), 0, s,
                       static_cast<const double*>(speed), n, flag);
  else
    hipLaunchKernelGGL(k_check_speeds<float>, dim3(b), dim3(kBlock), 0, s,
                       static_cast<const float*>(speed), n, flag);
  return hipGetLastError();
}

hipError_t dar_from_speeds(bool f64, int32_t n_paths, const int32_t* path_ptr,
                           const int32_t* path_link, int64_t n_pairs, int32_t L, const void* len,
                           const void* speed, int32_t n_days, int32_t H_speed, double dt, int32_t H,
                           int32_t K, void* traj, int32_t chunk, void* Rr, void* exit_time,
                           double* sums, void* cost, hipStream_t s) {
  if (f64)
    return run<double>(n_paths, path_ptr, path_link, n_pairs, L, static_cast<const double*>(len),
                       static_cast<const double*>(speed), n_days, H_speed, dt, H, K,
                       static_cast<double*>(traj), chunk, static_cast<double*>(Rr),
                       static_cast<double*>(exit_time), sums, static_cast<double*>(cost), s);
  return run<float>(n_paths, path_ptr, path_link, n_pairs, L, static_cast<const float*>(len),
                    static_cast<const float*>(speed), n_days, H_speed, static_cast<float>(dt), H, K,
                    static_cast<float*>(traj), chunk, static_cast<float*>(Rr),
                    static_cast<float*>(exit_time), sums, static_cast<float*>(cost), s);
}

int32_t dar_fused_patterns(bool f64, int32_t n_paths, int32_t longest, int32_t H, int32_t H_speed,
                           int32_t K) {
  const int seg = f64 ? (K <= 8 ? Seg<double, 8>::kLinks : Seg<double, 16>::kLinks)
                      : (K <= 8 ? Seg<float, 8>::kLinks : Seg<float, 16>::kLinks);
  if (longest > seg * kMaxSegs || H_speed > (1 << 24)) return 0;
  // a block per path and 63 intervals, a wave per segment of the longest path
  const int64_t threads =
      (int64_t)n_paths * (((int64_t)H + 62) / 63) * 64 * std::max(1, (longest + seg - 1) / seg);
  return (int32_t)std::min<int64_t>(kPatterns, kGridThreads / threads);
}

DarSplit dar_split(bool f64, int32_t n_paths, int64_t n_pairs, int32_t longest, int32_t H,
                   int32_t H_speed, int32_t K, int32_t n_patterns, const int32_t* pattern_ptr,
                   size_t limit) {
  DarSplit sp;
  sp.per_launch = dar_fused_patterns(f64, n_paths, longest, H, H_speed, K);
  if (sp.per_launch < 1) return sp;
  const int seg = f64 ? (K <= 8 ? Seg<double, 8>::kLinks : Seg<double, 16>::kLinks)
                      : (K <= 8 ? Seg<float, 8>::kLinks : Seg<float, 16>::kLinks);
  const int nd = f64 ? (K <= 8 ? Seg<double, 8>::kDays : Seg<double, 16>::kDays) : Seg<float, 8>::kDays;
  const size_t ss = f64 ? 8 : 4;
  const int64_t blocks = (int64_t)n_paths * (((int64_t)H + 62) / 63);   // of a pattern
  const int64_t segs = std::max(1, (longest + seg - 1) / seg) - 1;   // steps until the last one starts
  const size_t part_bytes = (size_t)H * ((size_t)K * n_pairs * ss + (size_t)n_paths * 8);
  limit = std::min(limit, size_t(64) << 20);
  // A block takes the days of its pattern one group after the other, and a group
  // passes through a segment of links after the other: us of a step, and of a call
  // of `steps` whose blocks fit the chip together.
  const double step_us = 1.5 * std::min(longest, seg) * (K > 8 ? 1.7 : 1.0);
  auto one_us = [&](int64_t steps) { return 80.0 + step_us * steps; };
  // The two kernels take links and days side by side, but the patterns in turn, and
  // trajectories have to be allocated.  Both models within 10 and 21% (standard
  // deviation) over 618 calls of 1 to 100 paths of 3 to 60 links, 8 to 1095 days in 1
  // and 4 patterns (120 days of one path of 60 links, 24 intervals, 12 lags, FP32:
  // 218 us in two kernels, 426 in one).
  auto two_pay = [&](int64_t steps, int64_t patterns, int64_t all_days, int64_t most) {
    const double mb = 1e-6 * n_pairs * (H + 1) * ss * most;
    return blocks * patterns <= 128 && mb <= 64.0 &&
           1.2 * (104.0 + 26.0 * patterns + (0.34 + 0.01 * longest) * all_days + 2.1 * mb) < one_us(steps);
  };
  // The groups of a pattern are split for two blocks per CU (one, if its segments make
  // more than four waves) as long as a part has more groups than the blocks have
  // segments to fill, and for up to 64 blocks down to four groups a part, where that
  // saves more than the parts' sums cost (whole calls with the splits, without, and in
  // the two kernels; 20 links, 288 intervals, FP32: 365 days, 1 path 207, 713 and 332
  // us, 10 paths 264, 718 and 647, 30 paths 404, 721 and 677, 50 paths 513, 721 and 816;
  // 1095 days, 10 paths 433, 1934 and 1122, in 4 patterns 374, 604 and 860).
  // The parts follow from the pattern's own days alone, so that it has the same
  // bits in a call of its own.
  int32_t most_parts = 1, most_days = 0;
  for (int32_t q = 0; q < n_patterns; ++q) {
    const int64_t days = pattern_ptr[q + 1] - pattern_ptr[q], groups = (days + nd - 1) / nd;
    int64_t parts = std::max(std::min(64 / blocks, groups / 4),
                             std::min((segs < 4 ? 512 : 256) / blocks,
                                      groups / std::max<int64_t>(4, segs)));
    parts = std::max<int64_t>(1, std::min<int64_t>(parts, limit / part_bytes));
    const int64_t steps = (groups + parts - 1) / parts;
    if (step_us * (groups - steps) < 50.0 + 6e-6 * part_bytes * parts ||   // sums, launch, allocation
        two_pay(steps + segs, 1, days, days))
      parts = 1;
    sp.parts.push_back((int32_t)parts);
    most_parts = std::max(most_parts, (int32_t)parts);
    most_days = std::max(most_days, (int32_t)days);
  }
  if (most_parts == 1) {
    if (two_pay((most_days + nd - 1) / nd + segs, n_patterns, pattern_ptr[n_patterns], most_days))
      sp.per_launch = 0;
    return sp;
  }
  sp.per_launch = (int32_t)std::min<int64_t>(sp.per_launch, limit / (most_parts * part_bytes));
  sp.scratch = std::min(sp.per_launch, n_patterns) * most_parts * part_bytes;
  return sp;
}

hipError_t dar_ratios(bool f64, int32_t n_paths, const int32_t* path_ptr, const int32_t* path_link,
                      int64_t n_pairs, int32_t longest, int32_t L, const void* len,
                      const void* speed, int32_t n_patterns, const int32_t* pattern_ptr,
                      int32_t H_speed, double dt, int32_t H, int32_t K, void* Rr, void* cost,
                      const DarSplit& split, void* scratch, hipStream_t s) {
  return f64 ? fused<double>(n_paths, path_ptr, path_link, n_pairs, longest, L, len, speed,
                             n_patterns, pattern_ptr, H_speed, dt, H, K, Rr, cost, split, scratch, s)
             : fused<float>(n_paths, path_ptr, path_link, n_pairs, longest, L, len, speed,
                            n_patterns, pattern_ptr, H_speed, dt, H, K, Rr, cost, split, scratch, s);
}
