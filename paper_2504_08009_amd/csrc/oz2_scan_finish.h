// Shared by the kernels that follow a stage 1 without atomics (oz2_stage1.hip): each of its workgroups reports in a slot
// of its own whether it saw an infinity or a NaN, and one workgroup of the next launch forms the flag word (1 when any
// slot is set) and clears the counters of the GEMM's round synchronisation.
#ifndef OZ2_SCAN_FINISH_H
#define OZ2_SCAN_FINISH_H

#include "oz2_internal.h"

// all threads of the workgroup
__device__ __forceinline__ void finish_scan(const Oz2ScanFinish& f) {
  int bad = 0;
  for (unsigned i = threadIdx.x; i < f.count; i += blockDim.x) bad |= f.slots[i] != 0ull;
  bad = __syncthreads_or(bad);
  if (threadIdx.x < 32) f.flags[threadIdx.x] = (threadIdx.x == 0 && bad) ? 1ull : 0ull;
}

#endif
