// First level of the strip reduction, shared by the profile's reduce
// (sas_kernels.hip) and the binned form's final sums (sas_bins.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "sas_kernels.hpp"
#include "sas_schedule.hpp"

namespace sas {

// Sums the strip rows of slice sl (256 threads; blockIdx.y the first group of
// 64 columns): see the reduce section of sas_kernels.hip for the order.
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
    if (m < Nq)
      for (int64_t t = a; t < b; ++t) acc += partial[t * Nq + m];
    __syncthreads();
    part[w][lane] = acc;
    __syncthreads();
    if (w == 0 && m < Nq) slice_sums[sl * Nq + m] = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
  }
}

}  // namespace sas
