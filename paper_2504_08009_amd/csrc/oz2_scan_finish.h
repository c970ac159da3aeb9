// Shared by the kernels that follow a stage 1 without atomics (oz2_stage1.hip): it reports in words of its own (see
// Oz2ScanFinish) whether it saw an infinity or a NaN, and one workgroup of the next launch forms the flag word (1 when any
// report is bad) and clears the counters of the GEMM's round synchronisation.  The other workgroups of that launch cannot
// look at the flag word yet; where it pays (oz2_stage2.hip) they look at the slots.
#ifndef OZ2_SCAN_FINISH_H
#define OZ2_SCAN_FINISH_H

#include "oz2_gemm.h"
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

__device__ __forceinline__ void write_flags(const Oz2ScanFinish& f, int bad) {
  if (threadIdx.x < 32) f.flags[threadIdx.x] = (threadIdx.x == 0 && bad) ? 1ull : 0ull;
}

// all threads of the workgroup
__device__ __forceinline__ void finish_scan(const Oz2ScanFinish& f) { write_flags(f, scan_found(f)); }

// The same look in a workgroup that is about to fetch its first tiles: the reports go to LDS ahead of them (`addr`: room for
// the words that nothing uses yet), so that who waits for the first tile has the reports too, and no load is waited for
// alone.  256 threads, wave wv of the four, lane lane.  Whole calls, us, no look / loads of their own behind the copies, one after the
// other where there are fewer than four per thread / this: 14 moduli 1000 x 1000 x 1500 50.8 / 52.4, 47.8 / 48.4, 1500^3 87.2 / 88.7,
// 82.8 / 83.3, dtrmm 1100 x 3000 118 / 123, 111.5 / 114; with an infinity 1000 x 1000 x 4000 1013 / 940.
__device__ __forceinline__ void fetch_reports(const Oz2ScanFinish& f, unsigned addr, int wv, int lane) {
  const int8_t* const from = reinterpret_cast<const int8_t*>(f.slots);
  for (unsigned c = wv; 128 * c < f.count; c += 4)  // 128 words per load; their number is even
    if (128 * c + 2 * lane < f.count) load_to_lds_16(from + 1024 * c, 16u * lane, addr + 1024 * c);
}
// all threads, after a barrier behind the wait for those loads; the room is free again when this returns
__device__ __forceinline__ int fetched_report_bad(const Oz2ScanFinish& f, const char* room) {
  typedef unsigned v4 __attribute__((ext_vector_type(4)));
  unsigned any = 0u;
  for (unsigned i = threadIdx.x; 2 * i < f.count; i += 256) {
    const v4 two = reinterpret_cast<const v4*>(room)[i];
    any |= two[1] | two[3];
  }
  return __syncthreads_or((int)any < 0);
}

#endif
