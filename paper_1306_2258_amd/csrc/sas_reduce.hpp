// The strip reduction, shared by the profile's reduce (sas_kernels.hip) and the
// binned form's final sums (sas_bins.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "sas_kernels.hpp"
#include "sas_schedule.hpp"

namespace sas {

// Sums the strip rows of slice sl (256 threads; blockIdx.y the first group of
// 64 columns): see the reduce section of sas_kernels.hip for the order.
// AGENT: the sums are stored past this XCD's cache, for a work-group of the same
// kernel to read.
template <bool AGENT = false>
__device__ __forceinline__ void reduce_slice(const DescView& sd, int64_t sl, const double* __restrict__ partial,
                                             int32_t Nq, double* __restrict__ slice_sums) {
  __shared__ double part[4][kWave];
  const int s = find_struct_by_slice(sd, sl);
  const StructDesc d = sd.get(s);
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int64_t first = d.strip_off + (sl - d.slice_off) * kSliceTiles;
  const int64_t last = min(first + kSliceTiles, d.strip_off + d.n_strips);
  constexpr int kQuarter = kSliceTiles / 4;
  const int64_t a = first + w * kQuarter, b = min(last, a + kQuarter);
  const int groups = static_cast<int>(ceil_div(Nq, kWave));
  for (int g = blockIdx.y; g < groups; g += gridDim.y) {  // (grid.y is capped at 65535)
    const int m = g * kWave + lane;
    double acc = 0.0;
    if (m < Nq) {
      // (sixteen loads in flight: one at a time took 20 us for 2,250 strips)
#pragma unroll 16
      for (int64_t t = a; t < b; ++t) acc += partial[t * Nq + m];
    }
    __syncthreads();
    part[w][lane] = acc;
    __syncthreads();
    if (w == 0 && m < Nq) {
      const double v = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
      if (AGENT)
        __hip_atomic_store(slice_sums + sl * Nq + m, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        slice_sums[sl * Nq + m] = v;
    }
  }
}

// A value of another work-group of the same kernel (AGENT), or of an earlier one.
template <bool AGENT>
__device__ __forceinline__ double read_sum(const double* p) {
  return AGENT ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}

// The profile of structure s at the 64 q values of group g (256 threads): wave w
// adds the slices w, w + 4, ... in order, the four sums are added in wave
// order, and Eq. 2's diagonal, the 2/q factor and the exact q = 0 value follow.
// With `rows` >= 0 the pair sums are complete and come as that many rows of
// partial profiles at `part` instead, added in order.
template <bool AGENT = false>
__device__ __forceinline__ void reduce_final(const DescView& sd, int s, int g, const double* __restrict__ slice_sums,
                                             const int32_t* __restrict__ toff, const double* __restrict__ asum,
                                             const float* __restrict__ table, int32_t T, int32_t Nq, double q0,
                                             double dq, const double* __restrict__ qdev, double* __restrict__ I_out,
                                             int rows = -1, const double* __restrict__ prows = nullptr) {
  __shared__ double part[4][kWave];
  const StructDesc d = sd.get(s);
  const int32_t* o = toff ? toff + static_cast<int64_t>(s) * (T + 1) : nullptr;
  const int64_t nb = ceil_div(d.n, kPackBlock);
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int m = g * kWave + lane;
  const bool vm = m < Nq;
  const double qm = vm ? (qdev ? qdev[m] : q0 + m * dq) : 1.0;
  double pairs = 0.0;
  if (vm && qm != 0.0) {
    if (rows >= 0) {
      // (by the first wave alone: one work-group that adds its own rows gives
      // the same sum)
      const int mine = w == 0 ? rows : 0;
#pragma unroll 16
      for (int k = 0; k < mine; ++k) pairs += read_sum<AGENT>(prows + static_cast<int64_t>(k) * Nq + m);
    } else {
#pragma unroll 8
      for (int64_t k = w; k < d.n_slices; k += 4) pairs += read_sum<AGENT>(slice_sums + (d.slice_off + k) * Nq + m);
    }
  }
  __syncthreads();
  part[w][lane] = pairs;
  __syncthreads();
  if (w == 0 && vm) {
    double val;
    if (qm == 0.0) {
      double f = 0.0;
      if (asum) {
#pragma unroll 16
        for (int64_t k = 0; k < nb; ++k) f += asum[((d.pack_off + k) * 2 + 0) * Nq + m];
      } else {
        for (int t = 0; t < T; ++t)
          f += static_cast<double>(o[t + 1] - o[t]) * static_cast<double>(table[static_cast<int64_t>(t) * Nq + m]);
      }
      val = f * f;
    } else {
      const double psum = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
      double diag = 0.0;
      if (asum) {
#pragma unroll 16
        for (int64_t k = 0; k < nb; ++k) diag += asum[((d.pack_off + k) * 2 + 1) * Nq + m];
      } else {
        for (int t = 0; t < T; ++t) {
          const double f = table[static_cast<int64_t>(t) * Nq + m];
          diag += static_cast<double>(o[t + 1] - o[t]) * f * f;
        }
      }
      val = rows >= 0 ? diag + psum : diag + (2.0 / qm) * psum;
    }
    I_out[static_cast<int64_t>(d.orig) * Nq + m] = val;
  }
}

}  // namespace sas
