// toep_hetero.hpp -- persistent pass of a plan's Toeplitz sensors: the row and
// column passes of all of them in one launch, claimed from a device counter like
// k_hetero's (same counters, dependency waits and error flag).  The bodies are
// those of the per-sensor launches, so both give the same bits.
// One workgroup of 256 lanes per CU: the largest tiles take the register file
// of one wave per SIMD.
#pragma once

#include "toep_persistent.hpp"

namespace pwfs {

// Set-up that does not depend on the claimed item stays in its own branch: the
// lane index is read from LDS after every claim (see k_hetero).
__global__ __launch_bounds__(256, 1) void k_toep_hetero(ToepHeteroArgs) {
  // read where the launch put them: indexed by sensor, a copy would go to scratch
  const ToepHeteroArgs& p = *(const ToepHeteroArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __align__(16) unsigned char toep_smem[];
  __shared__ int s_item, s_skip, s_zero;
  if (threadIdx.x == 0) s_zero = 0;
  for (;;) {
    if (threadIdx.x == 0) s_item = atomicAdd(&p.counters[0], 1);
    __syncthreads();
    int item = __builtin_amdgcn_readfirstlane(s_item);
    const int tid = (int)threadIdx.x + __builtin_amdgcn_readfirstlane(s_zero);
    __syncthreads();
    if (item >= p.total) break;
    int kind = 0, s = 0;
    for (kind = 0; kind < 2; ++kind) {
      bool found = false;
      for (int o = 0; o < p.n_sensors; ++o) {
        const int c = p.n_items[kind][p.order[o]];
        if (item < c) {
          s = p.order[o];
          found = true;
          break;
        }
        item -= c;
      }
      if (found) break;
    }
    kind = __builtin_amdgcn_readfirstlane(kind);
    s = __builtin_amdgcn_readfirstlane(s);
    item = __builtin_amdgcn_readfirstlane(item);
    bool skip = false;
    if (kind > 0) {
      if (threadIdx.x == 0) {
        int* dep = &p.counters[1 + s];
        const int need = p.n_items[0][s];
        int spins = 0, gave_up = p.spin_limit < 0;
        while (!gave_up && __hip_atomic_load(dep, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < need) {
          __builtin_amdgcn_s_sleep(2);
          if (++spins > p.spin_limit) gave_up = 1;
        }
        if (gave_up) atomicExch(p.flag, 1);
        s_skip = gave_up;
      }
      __syncthreads();
      skip = __builtin_amdgcn_readfirstlane(s_skip) != 0;
    }
    if (skip) {
      // the item's inputs may be incomplete: leave its outputs untouched
    } else if (kind == 0) {
      switch (p.ks[s]) {
        case 1: toep_rows_body<1>(p.rows[s], item, toep_smem, tid); break;
        case 2: toep_rows_body<2>(p.rows[s], item, toep_smem, tid); break;
        case 3: toep_rows_body<3>(p.rows[s], item, toep_smem, tid); break;
        case 4: toep_rows_body<4>(p.rows[s], item, toep_smem, tid); break;
        case 5: toep_rows_body<5>(p.rows[s], item, toep_smem, tid); break;
        case 6: toep_rows_body<6>(p.rows[s], item, toep_smem, tid); break;
        case 7: toep_rows_body<7>(p.rows[s], item, toep_smem, tid); break;
        default: toep_rows_body<8>(p.rows[s], item, toep_smem, tid); break;
      }
    } else {
      switch (p.ks[s]) {
        case 1: toep_cols_body<1, false>(p.cols[s], item, toep_smem, tid); break;
        case 2: toep_cols_body<2, false>(p.cols[s], item, toep_smem, tid); break;
        case 3: toep_cols_body<3, false>(p.cols[s], item, toep_smem, tid); break;
        case 4: toep_cols_body<4, false>(p.cols[s], item, toep_smem, tid); break;
        case 5: toep_cols_body<5, false>(p.cols[s], item, toep_smem, tid); break;
        case 6: toep_cols_body<6, false>(p.cols[s], item, toep_smem, tid); break;
        case 7: toep_cols_body<7, false>(p.cols[s], item, toep_smem, tid); break;
        default: toep_cols_body<8, false>(p.cols[s], item, toep_smem, tid); break;
      }
    }
    toep_landed();     // this wavefront's stores have reached the L2 ...
    __syncthreads();   // ... and every other's; the LDS is free
    if (threadIdx.x == 0 && kind == 0)
      __hip_atomic_fetch_add(&p.counters[1 + s], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

hipError_t toep_hetero_launch(const ToepHeteroArgs& a, int grid, size_t lds, hipStream_t st) {
  hipLaunchKernelGGL(k_toep_hetero, dim3((unsigned)grid), dim3(256), lds, st, a);
  return hipGetLastError();
}
void toep_hetero_limit() {
  if (hipFuncSetAttribute((const void*)k_toep_hetero, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024) !=
      hipSuccess)
    (void)hipGetLastError();
}

}  // namespace pwfs
