// Exceptional inputs (Section 3.1, closing remark): infinities and NaNs in A or B are detected in stage 1 (the row /
// column maxima are taken on bit patterns, where every non-finite value compares above every finite one) and the
// whole update C := alpha * op(A) * op(B) + beta * C is then formed in ordinary FP64 arithmetic (the tile routine
// of oz2_fallback_tile.h).  The kernel below is launched after stage 3 of a checked call and returns at once when
// the flag is clear, so the decision needs no device-to-host synchronisation; small problems carry its blocks in
// the launch of stage 3 instead.
#include "oz2_fallback_tile.h"
#include "oz2_internal.h"

namespace {

constexpr int kThreads = kFallbackThreads;

// (A few workgroups per compute unit walk the columns: with one per 256 elements the launch took 7 us to find that
// there is nothing to do at 4096 x 2048, now 4.)
__global__ void __launch_bounds__(kThreads) copy_if_kernel(const unsigned long long* __restrict__ flag, int64_t m, int64_t n,
                                                           const double* __restrict__ src, double* __restrict__ dst,
                                                           int64_t ld) {
  if (*flag == 0ull) return;
  for (int64_t j = blockIdx.x; j < n; j += gridDim.x)
    for (int64_t i = threadIdx.x; i < m; i += kThreads) dst[i + j * ld] = src[i + j * m];
}

__global__ void __launch_bounds__(kThreads) fp64_fallback_kernel(const unsigned long long* __restrict__ flag,
                                                                 const Oz2FallbackArgs f) {
  if (*flag == 0ull) return;
  oz2_fallback_tile<kFallbackTile>(f, (int64_t)blockIdx.x);
}

}  // namespace

hipError_t oz2_launch_fallback(const unsigned long long* flag, int transa, int transb, int64_t m, int64_t n, int64_t k,
                               double alpha, const double* A, int64_t lda, const double* B, int64_t ldb, double beta,
                               double* C, int64_t ldc, int triangle, int tri_a, int tri_b, hipStream_t st) {
  const int64_t tiles_m = (m + kFallbackTile - 1) / kFallbackTile, tiles_n = (n + kFallbackTile - 1) / kFallbackTile;
  if (tiles_m * tiles_n >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const Oz2FallbackArgs f = {transa, transb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, tiles_m, triangle, tri_a, tri_b};
  hipLaunchKernelGGL(fp64_fallback_kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(kThreads), 0, st, flag, f);
  return hipGetLastError();
}

hipError_t oz2_launch_copy_if(const unsigned long long* flag, int64_t m, int64_t n, const double* src, double* dst,
                              int64_t ld, hipStream_t st) {
  const dim3 grid((unsigned)(n < 1024 ? n : 1024));
  hipLaunchKernelGGL(copy_if_kernel, grid, dim3(kThreads), 0, st, flag, m, n, src, dst, ld);
  return hipGetLastError();
}
