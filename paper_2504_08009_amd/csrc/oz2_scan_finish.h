// Shared by the kernels that follow a stage 1 without atomics (oz2_stage1.hip): it reports in words of its own (see
// Oz2ScanFinish) whether it saw an infinity or a NaN, and one workgroup of the next launch forms the flag word (1 when any
// report is bad) and clears the counters of the GEMM's round synchronisation.  The other workgroups of that launch cannot
// look at the flag word yet; where it pays (oz2_stage2.hip) they look at the slots.
#ifndef OZ2_SCAN_FINISH_H
#define OZ2_SCAN_FINISH_H

#include "oz2_internal.h"

// all threads of the workgroup: is any report bad (its highest bit set)?
__device__ __forceinline__ int scan_found(const Oz2ScanFinish& f) {
  unsigned long long any = 0ull;
  unsigned i = threadIdx.x;
  for (; i + 3 * blockDim.x < f.count; i += 4 * blockDim.x) {
    unsigned long long v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = f.slots[i + u * blockDim.x];
    any |= v[0] | v[1] | v[2] | v[3];
  }
  for (; i < f.count; i += blockDim.x) any |= f.slots[i];
  return __syncthreads_or((long long)any < 0);
}

// all threads of the workgroup
__device__ __forceinline__ void finish_scan(const Oz2ScanFinish& f) {
  const int bad = scan_found(f);
  if (threadIdx.x < 32) f.flags[threadIdx.x] = (threadIdx.x == 0 && bad) ? 1ull : 0ull;
}

#endif
