// The device copies of one cluster's assignment values: the link-sliced W, the
// OD-sliced WT, the packed union tiles and the matrix-core tiles, all from one
// stored code per entry.
//
// One block per (lag, interval): it stages the block's codes in W's slot order
// in LDS (W itself where they do not fit), then writes the other copies line by
// line, each slot taking its code through an index (code_of: slot -> W slot, -1
// for padding).  Bound by the bytes written.  Every line is written whole, zeros
// included: scattering the entries into their places wrote a cache line per
// entry (the two sliced copies alone took 112 us in FP32 for 150 ODs, 500
// links, 288 intervals and 6 lags, 6000 entries per block).
#include "dode_internal.h"
#include "numfmt.h"

namespace {

constexpr int kBlock = 512;
// What a block may stage: a CU's LDS, as one block that gathers from it is faster
// than several that gather from memory (150 ODs, 500 links, 8% independent
// incidence in FP64, 92 KB: 233 us at three blocks' share of 48 KB, 150 us; 66 KB of
// a corridor the same 55 us).
constexpr size_t kStageBytes = 156 * 1024;

template <typename E>
struct alignas(4 * sizeof(E)) Four {
  E v[4];
};

template <int ST>
struct CodeT;
template <>
struct CodeT<DODE_F64> {
  using E = double;
  template <typename S>
  __device__ static E code(S w, float) { return static_cast<double>(w); }
};
template <>
struct CodeT<DODE_F32> {
  using E = float;
  template <typename S>
  __device__ static E code(S w, float) { return static_cast<float>(w); }
};
template <>
struct CodeT<DODE_BF16> {
  using E = uint16_t;
  template <typename S>
  __device__ static E code(S w, float) { return f32_to_bf16_rne(static_cast<float>(w)); }
};
template <>
struct CodeT<DODE_FP8_E4M3> {
  using E = uint8_t;
  template <typename S>
  __device__ static E code(S w, float sc) { return f32_to_e4m3_rne(static_cast<float>(w) / sc); }
};

// src: the cluster's values [K][T][nnz] (state type, CSR order), or nullptr
// when W already holds the codes.
template <int ST, typename S, bool STAGE>
__global__ void __launch_bounds__(kBlock)
k_install(DevPat pt, DevTiles tl, int32_t c, const S* __restrict__ src,
          DevVals dv, float* __restrict__ scale, const int32_t* __restrict__ code_of) {
  using E = typename CodeT<ST>::E;
  extern __shared__ __align__(16) unsigned char stage_mem[];
  const int lt = blockIdx.y * pt.T + blockIdx.x, tid = threadIdx.x;
  const int64_t blk = (int64_t)c * pt.K * pt.T + lt;
  const int n_ptile = dv.n_ptile;
  E* wb = static_cast<E*>(const_cast<void*>(dv.W)) + blk * pt.sr_len;
  E* st = STAGE ? reinterpret_cast<E*>(stage_mem) : wb;
  if (src) {
    const S* s = src + (int64_t)lt * pt.nnz;
    __shared__ float smax[64];
    if constexpr (ST == DODE_FP8_E4M3) {
      for (int i = tid; i < n_ptile; i += kBlock) smax[i] = 0.f;
      __syncthreads();
      for (int64_t j = tid; j < pt.nnz; j += kBlock) {
        const float a = fabsf(static_cast<float>(s[j]));
        atomicMax(reinterpret_cast<unsigned int*>(&smax[pt.col[j] >> 6]), __float_as_uint(a));
      }
      __syncthreads();
      for (int i = tid; i < n_ptile; i += kBlock)
        scale[blk * n_ptile + i] = smax[i] > 0.f ? smax[i] / 448.f : 1.f;
    }
    if constexpr (STAGE) {   // padding slots
      for (int64_t i = tid; i < pt.sr_len / 4; i += kBlock)
        reinterpret_cast<Four<E>*>(st)[i] = Four<E>{};
      __syncthreads();
    }
    for (int64_t j = tid; j < pt.nnz; j += kBlock) {
      float sc = 1.f;
      if constexpr (ST == DODE_FP8_E4M3) {
        const float m = smax[pt.col[j] >> 6];
        sc = m > 0.f ? m / 448.f : 1.f;
      }
      st[pt.sr_pos[j]] = CodeT<ST>::code(s[j], sc);
    }
  } else if constexpr (STAGE) {
    for (int64_t i = tid; i < pt.sr_len / 4; i += kBlock)
      reinterpret_cast<Four<E>*>(st)[i] = reinterpret_cast<const Four<E>*>(wb)[i];
  }
  __threadfence_block();
  __syncthreads();
  if (STAGE && src)
    for (int64_t i = tid; i < pt.sr_len / 4; i += kBlock)
      reinterpret_cast<Four<E>*>(wb)[i] = reinterpret_cast<const Four<E>*>(st)[i];
  const int4* idx = reinterpret_cast<const int4*>(code_of);
  auto fill = [&](const void* copy, int64_t len) {   // this block's part of a copy
    E* dst = static_cast<E*>(const_cast<void*>(copy)) + blk * len;
    for (int64_t i = tid; i < len / 4; i += kBlock) {
      const int4 k = idx[i];
      Four<E> o;
      o.v[0] = k.x < 0 ? E(0) : st[k.x];
      o.v[1] = k.y < 0 ? E(0) : st[k.y];
      o.v[2] = k.z < 0 ? E(0) : st[k.z];
      o.v[3] = k.w < 0 ? E(0) : st[k.w];
      reinterpret_cast<Four<E>*>(dst)[i] = o;
    }
    idx += len / 4;
  };
  fill(dv.WT, pt.sc_len);
  if (blockIdx.y + blockIdx.x >= (unsigned)pt.H) return;   // a block no product reads
  if (dv.PR) {
    fill(dv.PR, dv.pr_len);
    fill(dv.PC, dv.pc_len);
  }
  if (tl.Fv) {
    fill(tl.Fv, (int64_t)tl.kf_total * 512);
    fill(tl.Gv, (int64_t)tl.kg_total * 512);
  }
}

template <int ST, typename S>
hipError_t launch(const dode_dar* dar, int32_t c, const void* src, hipStream_t s) {
  using E = typename CodeT<ST>::E;
  const size_t stage = (size_t)dar->sr_len * sizeof(E);
  const bool fits = stage <= kStageBytes;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(dar->dims.T, dar->dims.K), dim3(kBlock), fits ? stage : 0, s,
                       dar->pat(), dar->tiles, c, static_cast<const S*>(src), dar->vals(),
                       dar->d_scale, dar->d_code_of);
  };
  if (fits)
    go(k_install<ST, S, true>);
  else
    go(k_install<ST, S, false>);
  return hipGetLastError();
}

}  // namespace

hipError_t install_values(const dode_dar* dar, int32_t cluster, const void* W_state,
                          hipStream_t s) {
  switch (dar->storage) {
    case DODE_F64: return launch<DODE_F64, double>(dar, cluster, W_state, s);
    case DODE_F32: return launch<DODE_F32, float>(dar, cluster, W_state, s);
    case DODE_BF16: return launch<DODE_BF16, float>(dar, cluster, W_state, s);
    default: return launch<DODE_FP8_E4M3, float>(dar, cluster, W_state, s);
  }
}
