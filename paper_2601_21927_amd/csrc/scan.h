// Workgroup-wide prefix sums built from wave ballots (flags) and lane shifts (integers).
#pragma once

#include "common.h"

namespace sonic {

// Number of lanes below this one whose predicate is set.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
}

// Inclusive sum over the lanes of a wave, without LDS round trips: four shifts inside the
// rows of 16 lanes, then the rows' totals broadcast to the rows behind.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Exclusive prefix count of a 0/1 flag over an NT-thread workgroup.
// `lds` must hold NT/64 + 1 ints; the workgroup total is returned in *total.
template <int NT>
__device__ __forceinline__ int block_flag_scan(bool flag, int *total, int *lds) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  const uint64_t m = __ballot(flag);
  const int below = lanes_below(m);
  if (lane == 0) lds[w] = __popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < NW; ++i) {
      const int c = lds[i];
      lds[i] = run;
      run += c;
    }
    lds[NW] = run;
  }
  __syncthreads();
  const int res = lds[w] + below;
  *total = lds[NW];
  __syncthreads();
  return res;
}

// Exclusive prefix sums of NV ints at once over an NT-thread workgroup: below[f] =
// the sum of x[f] over lower threads, total[f] = the workgroup's sum.  Two barriers.
template <int NT, int NV>
__device__ __forceinline__ void block_int_scan_n(const int (&x)[NV], int (&below)[NV], int (&total)[NV],
                                                 int *lds) {
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  const int w = threadIdx.x / kWave;
  int v[NV];
#pragma unroll
  for (int f = 0; f < NV; ++f) v[f] = wave_scan(x[f]);
  if (lane == kWave - 1)
#pragma unroll
    for (int f = 0; f < NV; ++f) lds[f * NW + w] = v[f];
  lds_barrier();
#pragma unroll
  for (int f = 0; f < NV; ++f) {
    int before = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const int c = lds[f * NW + k];
      before += k < w ? c : 0;
      tot += c;
    }
    below[f] = v[f] - x[f] + before;
    total[f] = tot;
  }
  lds_barrier();
}

// Exclusive prefix sum of an int over an NT-thread workgroup.
template <int NT>
__device__ __forceinline__ int block_int_scan(int x, int *total, int *lds) {
  const int v[1] = {x};
  int below[1], tot[1];
  block_int_scan_n<NT, 1>(v, below, tot, lds);
  *total = tot[0];
  return below[0];
}

}  // namespace sonic
