// Kernel arguments on their way into the scalar cache.  Every launch finds its arguments in memory that no cache holds yet; a
// loop that reads one modulus' constants after the other out of them waits for a miss of the scalar cache, most of a
// microsecond, whenever it comes to new lines.  One word of every line, all loads in flight together, costs one such wait.
// Kernels that run for less than about ten microseconds gain (whole calls, us, without / with it: 14 moduli 64^3 14.5 / 12.7,
// 256^3 18.2 / 15.3, 512^3 23.9 / 22.7, 15 moduli 333 x 517 x 291 22.5 / 21.5, dsyrk 500 x 300 26.2 / 24.6); in the conversion of
// longer vectors, whose first workgroups have filled the cache for all others, it does not (1000 x 1000 x 1500 73.2 / 73.7).
#ifndef OZ2_WARM_H
#define OZ2_WARM_H

#include <hip/hip_runtime.h>

// `args`: a by-value argument of the kernel.  Uniform over the workgroup; near the start of the kernel.
template <class T>
__device__ __forceinline__ void warm_arguments(const T& args) {
  static_assert(sizeof(T) % 4 == 0, "words");
  const unsigned* p = reinterpret_cast<const unsigned*>(&args);
  unsigned x = p[sizeof(T) / 4 - 1];
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 4; i += 16) x |= p[i];  // 64-byte lines
  asm volatile("" ::"s"(x));
}

#endif
