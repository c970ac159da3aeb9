#ifndef OZ2_FAST_DIV_H
#define OZ2_FAST_DIV_H

#include <hip/hip_runtime.h>
#include <stdint.h>

// Division of numbers below 2^31 by one that the host knows: with s = 31 + ceil(log2 d) and m = ceil(2^s / d),
// n m / 2^s exceeds n / d by less than 1 / d.  On the device a scalar multiplication and a shift; the compiler's own
// division goes through the vector units' FP32 reciprocal, some thirty instructions per quotient that a workgroup
// would wait for between two tiles.
struct FastDiv {
  unsigned m, s;
};
inline FastDiv fast_div(unsigned d) {
  unsigned log = 0;
  while (((uint64_t)1 << log) < d) ++log;
  return {(unsigned)((((uint64_t)1 << (31 + log)) + d - 1) / d), 31 + log};
}
__device__ __forceinline__ int operator/(int n, const FastDiv& d) {
  return (int)(((uint64_t)(unsigned)n * d.m) >> d.s);
}

#endif
