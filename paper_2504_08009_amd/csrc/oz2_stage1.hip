// Stage 1 of Ozaki scheme II on gfx950: Algorithm 1 lines 1-5.
//   1a  per-row maximum of |A| and per-column maximum of |B| (bit patterns, 64-bit atomic max)
//   1a' shifts  sa_i = kappa - 1 - floor(log2 max_l |a_il|),  sb_j likewise  (Section 3, D and E); or, in the
//       modes of Section 4.1, from an integer bound of the 2-norms (one more pass over vectors that do not fit into LDS) or from the
//       row / column maxima of an INT8 product of 6-bit upper bounds of |A| and |B| (bound planes, one GEMM
//       launch, one pass over the product)
//   1b  a' = trunc(a * 2^sa_i) and its symmetric residues modulo every p_t, written as INT8 planes in the
//       blocked layout the GEMM reads (256 rows x 64 inner-dimension bytes per contiguous block), zero
//       padded up to the GEMM tile sizes.
// All are bound by HBM traffic: 8 bytes read per element in 1a, 8 read + N written in 1b.  The operands are far
// larger than the caches and every plane byte is written once, so loads and stores are non-temporal (measured:
// 3-6 % on stage 1).
// Infinities and NaNs are noticed in 1a (their bit patterns are above every finite magnitude) and recorded in
// a flag word of the workspace.  Triangular operands (TRMM shape) are masked while they are read.
// The maxima of both operands share one launch and so do their conversions (small problems are bound by the
// number of launches); a block picks its operand and its kernel body by its index.
#include <type_traits>

#include "oz2_math.h"
#include "oz2_bound.h"
#include "oz2_route.h"
#include "oz2_scan_finish.h"
#include "oz2_warm.h"

namespace {

constexpr int kThreads = 256;
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

__global__ void __launch_bounds__(kThreads) fill_u64_kernel(unsigned long long* p, int64_t count) {
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < count) p[i] = 0ull;
}

// Bit pattern of +infinity: as unsigned integers the magnitudes of infinities and NaNs are the values at or
// above it, every finite magnitude is below.
constexpr unsigned long long kInfBits = 0x7ff0000000000000ull;

// Triangular operands (TRMM shape): the array holds only one triangle; the rest is not referenced and counts
// as zero, the diagonal as one when it is declared unit.  (r, c) = row and column of the element in the
// stored array.  tri & 3: 0 = full matrix, 1 = lower (r >= c stored), 2 = upper (r <= c); tri & 4: unit diagonal.
__device__ __forceinline__ double tri_value(double v, int64_t r, int64_t c, int tri) {
  if (tri == 0) return v;
  if (r == c) return (tri & 4) ? 1.0 : v;
  const bool stored = (tri & 3) == 1 ? r > c : r < c;
  return stored ? v : 0.0;
}

__device__ __forceinline__ unsigned long long abs_bits(double v) {
  return (unsigned long long)__double_as_longlong(v) & 0x7fffffffffffffffull;
}

// A is m x k column-major: lanes run along rows (coalesced), each block covers 256 rows x KC columns.
constexpr int kRowMaxKC = 128;
__device__ __forceinline__ void strided_max(const double* __restrict__ A, int64_t lda, int64_t m, int64_t k,
                                            unsigned long long* __restrict__ rowmax,
                                            unsigned long long* __restrict__ nonfinite, int tri, unsigned bx,
                                            unsigned by) {
  int64_t i = (int64_t)bx * kThreads + threadIdx.x;
  if (i >= m) return;
  int64_t l0 = (int64_t)by * kRowMaxKC;
  int64_t l1 = l0 + kRowMaxKC < k ? l0 + kRowMaxKC : k;
  const double* p = A + i + l0 * lda;
  unsigned long long mx = 0ull;
  int64_t l = l0;
  for (; l + 8 <= l1; l += 8) {
    unsigned long long v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = abs_bits(tri_value(__builtin_nontemporal_load(p + (int64_t)u * lda), i, l + u, tri));
#pragma unroll
    for (int u = 0; u < 8; ++u) mx = v[u] > mx ? v[u] : mx;
    p += 8 * lda;
  }
  for (; l < l1; ++l) {
    unsigned long long v = abs_bits(tri_value(*p, i, l, tri));
    mx = v > mx ? v : mx;
    p += lda;
  }
  if (mx) atomicMax(rowmax + i, mx);
  if (mx >= kInfBits) *nonfinite = 1ull;
}

// B is k x n column-major: one block per (column, chunk of KC rows); lanes run down the column.
constexpr int kColMaxKC = 4096;
__device__ __forceinline__ void contig_max(const double* __restrict__ B, int64_t ldb, int64_t k,
                                           unsigned long long* __restrict__ colmax,
                                           unsigned long long* __restrict__ nonfinite, int tri, unsigned bx, unsigned by) {
  int64_t j = bx;
  int64_t l0 = (int64_t)by * kColMaxKC;
  const double* p = B + j * ldb;
  unsigned long long mx = 0ull;
#pragma unroll 4
  for (int u = 0; u < kColMaxKC / kThreads; ++u) {
    int64_t l = l0 + (int64_t)u * kThreads + threadIdx.x;
    if (l < k) {
      unsigned long long v = abs_bits(tri_value(__builtin_nontemporal_load(p + l), l, j, tri));
      mx = v > mx ? v : mx;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    unsigned long long o = __shfl_xor(mx, off, 64);
    mx = o > mx ? o : mx;
  }
  __shared__ unsigned long long part[kThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) mx = part[w] > mx ? part[w] : mx;
    if (mx) atomicMax(colmax + j, mx);
    if (mx >= kInfBits) *nonfinite = 1ull;
  }
}

// Both operands of a call in one launch: a block belongs to the first job or to the second by its index.
// strided: the vectors are rows of a column-major array (lanes along the vectors); otherwise they are its
// columns (lanes along the inner dimension).  gx: extent of the job's first (fast) block coordinate.
struct MaxJob {
  const double* X;
  int64_t ld, nvec, k;
  unsigned long long* vmax;
  int tri, strided;
  unsigned gx, nblk;
};
__global__ void __launch_bounds__(kThreads) operand_max_kernel(const MaxJob ja, const MaxJob jb,
                                                               unsigned long long* __restrict__ nonfinite) {
  const bool first = blockIdx.x < ja.nblk;
  const MaxJob& j = first ? ja : jb;
  const unsigned id = first ? blockIdx.x : blockIdx.x - ja.nblk;
  const unsigned bx = id % j.gx, by = id / j.gx;
  if (j.strided)
    strided_max(j.X, j.ld, j.nvec, j.k, j.vmax, nonfinite, j.tri, bx, by);
  else
    contig_max(j.X, j.ld, j.k, j.vmax, nonfinite, j.tri, bx, by);
}

// ---- Cauchy-Schwarz shift mode (Section 4.1): integer upper bound of the 2-norm.
// With e = floor(log2 max |x|):  q_l = ceil(|x_l| 2^(19-e)) <= 2^20,  S = sum_l q_l^2  (exact in 64 bits for
// fewer than 2^23 terms, and independent of the order of summation).
__device__ __forceinline__ int exponent_of_bits(unsigned long long b) {  // floor(log2) of a positive double's bits
  int be = (int)(b >> 52);
  return be ? be - 1023 : (63 - __clzll((long long)b)) - 1074;
}

__device__ __forceinline__ double scaled_ceil_sq(double v, int sc) {
  double q = ceil(ldexp(fabs(v), sc));  // exact: a power-of-two scaling, then an integer at most 2^20
  if (v != 0.0 && q == 0.0) q = 1.0;    // the scaling underflowed: the ceiling of a positive value is 1
  return q * q;                         // exact: at most 2^40
}

__global__ void __launch_bounds__(kThreads) rownorm_kernel(const double* __restrict__ A, int64_t lda, int64_t m,
                                                           int64_t k, const unsigned long long* __restrict__ rowmax,
                                                           unsigned long long* __restrict__ rownorm, int tri) {
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= m) return;
  const unsigned long long mb = rowmax[i];
  if (!mb) return;
  const int sc = 19 - exponent_of_bits(mb);
  int64_t l0 = (int64_t)blockIdx.y * kRowMaxKC;
  int64_t l1 = l0 + kRowMaxKC < k ? l0 + kRowMaxKC : k;
  const double* p = A + i + l0 * lda;
  double acc = 0.0;  // at most 128 terms of at most 2^40: exact
  int64_t l = l0;
  for (; l + 8 <= l1; l += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = tri_value(p[(int64_t)u * lda], i, l + u, tri);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += scaled_ceil_sq(v[u], sc);
    p += 8 * lda;
  }
  for (; l < l1; ++l) {
    acc += scaled_ceil_sq(tri_value(*p, i, l, tri), sc);
    p += lda;
  }
  atomicAdd(rownorm + i, (unsigned long long)acc);
}

__global__ void __launch_bounds__(kThreads) colnorm_kernel(const double* __restrict__ B, int64_t ldb, int64_t k,
                                                           const unsigned long long* __restrict__ colmax,
                                                           unsigned long long* __restrict__ colnorm, int tri) {
  int64_t j = blockIdx.x;
  const unsigned long long mb = colmax[j];
  if (!mb) return;  // uniform over the block
  const int sc = 19 - exponent_of_bits(mb);
  int64_t l0 = (int64_t)blockIdx.y * kColMaxKC;
  const double* p = B + j * ldb;
  double acc = 0.0;  // 16 terms
#pragma unroll 4
  for (int u = 0; u < kColMaxKC / kThreads; ++u) {
    int64_t l = l0 + (int64_t)u * kThreads + threadIdx.x;
    if (l < k) acc += scaled_ceil_sq(tri_value(p[l], l, j, tri), sc);
  }
  unsigned long long s = (unsigned long long)acc;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  __shared__ unsigned long long part[kThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) s += part[w];
    atomicAdd(colnorm + j, s);
  }
}

// Shifts of both operands in one launch (Algorithm 1 line 1).  Per vector, from the bit pattern b of its largest
// magnitude (e = floor(log2) of it) and, in the modes of Section 4.1, a second quantity v:
//   mode 0 (Section 3):       kappa - 1 - e                         (param = kappa)
//   mode 1 (Cauchy-Schwarz):  beta - (e - 19 + h), h = min{h : 4^h >= v}, v = integer norm bound S >= 2^38  (param = beta)
//   mode 2 (INT8 product):    floor((b2 - t)/2) - (e - 5), t = min{t : 2^t >= v}, v = largest element of the bound
//                             product in the vector's row / column      (param = b2)
// An all-zero vector gets shift 0.
// With unequal bit budgets (Section 3: k_A != k_B when the operands differ in precision) each operand has its
// own param (modes 0, 1) or an offset added at the end (mode 2).
__device__ __forceinline__ int shift_of(unsigned long long b, unsigned long long v, int mode, int param, int offset) {
  if (!b) return 0;
  const int e = exponent_of_bits(b);
  if (mode == 0) return param - 1 - e;
  if (mode == 1) {
    const int bits = 64 - __clzll((long long)(v - 1));  // ceil(log2 S)
    return param - (e - 19 + ((bits + 1) >> 1));
  }
  if (!v) return 0;
  const int t = v <= 1 ? 0 : 64 - __clzll((long long)(v - 1));
  const int d = param - t;
  return (d >= 0 ? d / 2 : -((1 - d) / 2)) + offset - (e - 5);
}
struct ShiftJob {
  const unsigned long long* mx;
  const unsigned long long* aux;
  int* s;
  int64_t count;
  int param;
  int offset;
};
__global__ void __launch_bounds__(kThreads) shifts_kernel(const ShiftJob ja, const ShiftJob jb, int mode) {
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const bool first = i < ja.count;
  const ShiftJob& j = first ? ja : jb;
  if (!first) i -= ja.count;
  if (i >= j.count) return;
  j.s[i] = shift_of(j.mx[i], mode == 0 ? 0ull : j.aux[i], mode, j.param, j.offset);
}

// ---- Operands whose vectors are too long for the one-pass conversion (below): maxima, in the Cauchy-Schwarz mode the norm bounds, and shifts of both in ONE launch and
// without atomics, so that nothing has to be cleared first: a workgroup owns 16 whole vectors, forms their maxima (and
// from them, reading the vectors once more out of the caches, the sums of squares), writes them and the shifts, and reports
// in a slot of its own whether it saw an infinity or a NaN.  The conversion launch that follows folds the slots into the
// flag word.  Three launches fewer than fill + maxima + shifts, six with the norms; used while the operands are small
// enough that 16 vectors per workgroup still fill the chip.
// A triangular operand is read over the inner positions its 16 vectors can have, half of the array.
// Bound by the latency of the loads in flight.  Whole calls against separate launches (us): Cauchy-Schwarz mode, 14 moduli,
// 500^3 51 -> 40, 2048^3 212 -> 190, INT8-product mode 2048^3 277 -> 262; triangular product 4096 x 2048 of order 4096
// (with the conversion below, which leaves out the same half) 590 -> 480.
// 512 threads for the 16 vectors: twice the loads in flight where the workgroups are few (256 / 512 / 1024 threads, us: 500^3
// Cauchy-Schwarz 39.9 / 36.0 / 34.0, 1000 x 1000 x 2000 86.2 / 78.3 / 78.7, 256 x 256 x 4096 64.3 / 56.5 / 57.6, 300 x 3000 x 5000
// 258 / 246 / 251, 4096^3 1153 / 1151 / 1150).
constexpr int kScanVecs = 16;
constexpr int kScanThreads = 512;
struct ScanJob {
  const double* X;
  int64_t ld, nvec, nvec_pad, k;
  unsigned long long* vmax;
  unsigned long long* vnorm;  // norm bounds (mode 1), else cleared (the INT8-product mode gathers its maxima there)
  int* shifts;
  int param;  // as in ShiftJob
  int tri, strided;
  unsigned nblk;
};

// f(value) over this thread's share of vector v, element (v, l) at p[l * step], l = l0 .. l1 - 1 in strides; (r, c) of an
// element in the stored array: (v, l) or, when swapped, (l, v)
template <int STRIDE, class F>
__device__ __forceinline__ void walk_vector(const double* p, int64_t step, int64_t v, int64_t l0, int64_t l1, int tri, bool swapped,
                                            F&& f) {
  int64_t l = l0;
  for (; l + 7 * STRIDE < l1; l += 8 * STRIDE) {
    double x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = p[(l + u * STRIDE) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t lu = l + u * STRIDE;
      f(swapped ? tri_value(x[u], lu, v, tri) : tri_value(x[u], v, lu, tri));
    }
  }
  for (; l < l1; l += STRIDE) f(swapped ? tri_value(p[l * step], l, v, tri) : tri_value(p[l * step], v, l, tri));
}

__global__ void __launch_bounds__(kScanThreads) vector_scan_kernel(const ScanJob ja, const ScanJob jb, const int mode,
                                                               unsigned long long* __restrict__ slots) {
  constexpr int kEach = kScanVecs / (kScanThreads / 64);  // vectors a wave takes when they are columns
  constexpr int kPhases = kScanThreads / kScanVecs;
  __shared__ unsigned long long part[kScanThreads];
  __shared__ unsigned long long top[kScanVecs];
  const bool first = blockIdx.x < ja.nblk;
  const ScanJob& j = first ? ja : jb;
  const unsigned id = first ? blockIdx.x : blockIdx.x - ja.nblk;
  const int64_t v0 = (int64_t)id * kScanVecs;
  // inner positions a stored element of these vectors can have
  const bool swapped = !j.strided;  // the vectors are columns of the stored array
  int64_t lo = 0, hi = j.k;
  if (j.tri & 3) {
    const bool upto = ((j.tri & 3) == 1) != swapped;
    if (upto)
      hi = v0 + kScanVecs < hi ? v0 + kScanVecs : hi;
    else
      lo = v0 < hi ? v0 : hi;
  }
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // strided: element (v, l) at X[v + l ld]; 16 lanes along the vectors (128 contiguous bytes), kPhases along them.
  // otherwise: element (v, l) at X[l + v ld]; a wave takes kEach vectors in turn, its lanes run down the vector.
  const int vv = threadIdx.x & (kScanVecs - 1);
  // one value per vector in top[]: f(element, partial, vector) over a thread's share, then the partials joined
  auto reduce = [&](auto zero, auto&& f, auto&& join) {
    if (j.strided) {
      auto own = zero;
      const int64_t v = v0 + vv;
      if (v < j.nvec)
        walk_vector<kPhases>(j.X + v, j.ld, v, lo + threadIdx.x / kScanVecs, hi, j.tri, false, [&](double x) { own = f(x, own, vv); });
      unsigned long long acc = (unsigned long long)own;
      part[threadIdx.x] = acc;
      __syncthreads();
      if (threadIdx.x < kScanVecs) {
#pragma unroll
        for (int ph = 1; ph < kPhases; ++ph) acc = join(acc, part[threadIdx.x + ph * kScanVecs]);
        top[threadIdx.x] = acc;
      }
    } else {
#pragma unroll 1
      for (int q = 0; q < kEach; ++q) {
        const int w = wv * kEach + q;
        const int64_t v = v0 + w;
        auto own = zero;
        if (v < j.nvec) walk_vector<64>(j.X + v * j.ld, 1, v, lo + lane, hi, j.tri, true, [&](double x) { own = f(x, own, w); });
        unsigned long long acc = (unsigned long long)own;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc = join(acc, __shfl_xor(acc, off, 64));
        if (lane == 0) top[w] = acc;
      }
    }
    __syncthreads();
  };
  reduce(
      0ull,
      [](double x, unsigned long long own, int) {
        const unsigned long long b = abs_bits(x);
        return b > own ? b : own;
      },
      [](unsigned long long a, unsigned long long b) { return a > b ? a : b; });
  const unsigned long long mx = threadIdx.x < kScanVecs ? top[threadIdx.x] : 0ull;
  unsigned long long norm = 0ull;
  if (mode == 1) {
    __shared__ int scale[kScanVecs];
    if (threadIdx.x < kScanVecs) scale[threadIdx.x] = mx ? 19 - exponent_of_bits(mx) : 0;
    __syncthreads();
    // (a thread's sum is exact: at most 2^25 elements in at least 256 padded vectors, so vectors of at most 2^17 elements, of which a
    // thread adds at most 2^17 / kPhases = 2^12 terms of at most 2^40)
    static_assert(kPhases >= 32, "2^12 terms of a vector of 2^17 elements");
    reduce(0.0, [&](double x, double own, int w) { return own + scaled_ceil_sq(x, scale[w]); },
           [](unsigned long long a, unsigned long long b) { return a + b; });
    norm = threadIdx.x < kScanVecs ? top[threadIdx.x] : 0ull;
  }
  // threads 0 .. 15 hold the values of the 16 vectors
  bool bad = false;
  if (threadIdx.x < kScanVecs) {
    const int64_t v = v0 + threadIdx.x;
    if (v < j.nvec_pad) {
      j.vmax[v] = mx;
      j.vnorm[v] = norm;
      j.shifts[v] = shift_of(mx, norm, mode, j.param, 0);
    }
    bad = mx >= kInfBits;
  }
  const int any = __syncthreads_or(bad ? 1 : 0);
  if (threadIdx.x == 0) slots[blockIdx.x] = any ? kBadReport : 0ull;
}

__device__ __forceinline__ unsigned pack4(int r0, int r1, int r2, int r3) {
  return (unsigned)(r0 & 0xff) | ((unsigned)(r1 & 0xff) << 8) | ((unsigned)(r2 & 0xff) << 16) | ((unsigned)r3 << 24);
}

// sixteen consecutive inner-dimension values of one vector -> sixteen bound bytes
__device__ __forceinline__ void store_bounds(const double* mine, int shift, int8_t* dst) {
  int r[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) r[u] = oz2_bound6(mine[u], shift);
  uint4 v;
  v.x = pack4(r[0], r[1], r[2], r[3]);
  v.y = pack4(r[4], r[5], r[6], r[7]);
  v.z = pack4(r[8], r[9], r[10], r[11]);
  v.w = pack4(r[12], r[13], r[14], r[15]);
  *reinterpret_cast<uint4*>(dst) = v;
}

// ---- INT8-product shift mode (Section 4.1): row and column maxima of P = A''B'' (INT32, element (i,j) at
// j*m_pad + i).  A wave takes 256 rows (four per lane, 16-byte loads) x 8 to 64 columns; the four rows of a lane are joined
// before the wave's reduction, which is what the kernel spends its time on (3001 x 2777: 38 -> 27 us).  Few columns per wave are a
// short chain (64 against 8, whole calls with 16 moduli, us: 64^3 53.0 / 35.8, 200 x 300 x 700 68.3 / 51.0, 1000 x 1000 x 2000 136.4 / 125.8)
// but many waves that meet at a row's word (300 x 5000 x 700 134 / 157).
constexpr int kProdRows = kThreads / 64 * 256;
__global__ void __launch_bounds__(kThreads) prodmax_kernel(const int* __restrict__ P, int64_t m_pad, int64_t m, int64_t n,
                                                           int64_t row_blocks, int cols, unsigned long long* __restrict__ rowtop,
                                                           unsigned long long* __restrict__ coltop) {
  typedef int v4s __attribute__((ext_vector_type(4)));
  const int64_t rb = blockIdx.x % row_blocks, cb = blockIdx.x / row_blocks;
  const int lane = threadIdx.x & 63;
  const int64_t i = rb * kProdRows + (threadIdx.x >> 6) * 256 + 4 * lane;
  if (i - 4 * lane >= m_pad) return;  // the whole wave; m_pad is a multiple of 256
  const int64_t j0 = cb * cols;
  const int* src = P + i + j0 * m_pad;
  v4s rmax = {0, 0, 0, 0};
  for (int jj = 0; jj < cols; jj += 8) {
    v4s v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = j0 + jj + u < n ? __builtin_nontemporal_load(reinterpret_cast<const v4s*>(src + (int64_t)(jj + u) * m_pad)) : v4s{0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      // (rows beyond m are padding: zero operands, zero products)
      rmax = __builtin_elementwise_max(rmax, v[u]);
      int c = max(max(v[u].x, v[u].y), max(v[u].z, v[u].w));
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        int o = __shfl_xor(c, off, 64);
        c = o > c ? o : c;
      }
      if (lane == 0 && c > 0) atomicMax(coltop + j0 + jj + u, (unsigned long long)c);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (i + r < m && rmax[r] > 0) atomicMax(rowtop + i + r, (unsigned long long)rmax[r]);
}

// Plane layout (shared with the GEMM kernel): blocks of 256 rows x 64 bytes of the inner dimension, each
// block contiguous; element (row, l) of plane t at
//   ((t*rows_pad + 256*(row/256)) * k_pad) + (l/64)*16384 + (row%256)*64 + (l%64).
constexpr int kBlkRows = OZ2_TILE_M;   // 256
constexpr int kBlkK = OZ2_TILE_K;      // 64
static_assert(OZ2_TILE_M == 256 && OZ2_TILE_N == 256 && OZ2_TILE_K == 64, "plane layout is 256 x 64 blocks");

// A triangular operand (TRMM shape): do the products read inner positions l0 .. l1 - 1 of the block of 256 vectors that
// vector v0 belongs to?  They walk the k-tiles up to (upto) or from the diagonal block; what they leave out is not written.
__device__ __forceinline__ bool tile_used(int64_t v0, int64_t l0, int64_t l1, bool upto, int tri) {
  const int64_t d0 = v0 / kBlkRows * kBlkRows;
  return (tri & 3) == 0 || (upto ? l0 < d0 + kBlkRows : l1 > d0);
}

// A (m x k column-major) -> planes.  Block: 64 rows x 64 columns.  Every column segment (64 rows, 512
// bytes) is read coalesced with lanes along the rows, transposed through LDS so that a thread holds 16
// consecutive inner-dimension values of one row, and wave w writes, for every plane, the 1 KiB that its 16
// rows x 64 bytes occupy contiguously in the output block.
constexpr int kConvARows = 64;
constexpr int kConvAPitch = 65;  // doubles per row in LDS
// KIND 0 / 1: residues of trunc(a 2^shift) with the one- / two-level split; KIND 2: the single plane of 6-bit
// upper bounds ceil(|a| 2^shift) of Section 4.1 (written where plane 0 goes).
// KIND 3: the two-level split, its residues in the lean form.  Sixteen elements per thread take 165 registers and three waves per
// SIMD in the usual form, 122 and four in the lean one, which has two FP64 instructions more: the better one where the
// operands stream from memory, not where a call is a chain of latencies (stage 1, us, usual / lean: 22 moduli 176 x 10067 x 24807
// 2340 / 2087, 24 moduli 2653 x 6427 x 30545 2747 / 2434, 96 x 8192 x 8192 658 / 584, 22 moduli 4096^3 226 / 233, 2048^3 64 / 67).
template <int KIND>
__device__ __forceinline__ oz2_u16x2 conversion_residues(const Oz2SplitPair<(KIND & 1) != 0>& s, const Oz2ConvMod& m) {
  if constexpr (KIND == 3)
    return oz2_residue_pair_lean<true>(s, m);
  else
    return oz2_residue_pair<KIND == 1>(s, m);
}
template <int KIND>
__device__ __forceinline__ void convert_strided(const double* __restrict__ A, int64_t lda, int64_t m, int64_t k,
                                                int64_t m_pad, int64_t k_pad, const int* __restrict__ sa,
                                                int8_t* __restrict__ planes, const int tri, const bool cached,
                                                const Oz2ConvConsts& cc, double* tile, unsigned bx, unsigned by) {
  const int64_t r0 = (int64_t)bx * kConvARows;  // < m_pad
  const int64_t kb = by;
  if (KIND != 2 && !tile_used(r0, kb * kBlkK, kb * kBlkK + kBlkK, (tri & 3) == 1, tri)) return;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  {
    const int64_t i = r0 + lane;
    const double* src = A + i;
    auto read = [&](auto load) {
#pragma unroll 4
      for (int c = 0; c < kBlkK / 4; ++c) {
        const int lc = c * 4 + wv;
        const int64_t l = kb * kBlkK + lc;
        double v = (i < m && l < k) ? tri_value(load(src + l * lda), i, l, tri) : 0.0;
        tile[lane * kConvAPitch + lc] = v;
      }
    };
    if (cached)
      read([](const double* p) { return *p; });
    else
      read([](const double* p) { return __builtin_nontemporal_load(p); });
  }
  __syncthreads();
  const int row = wv * 16 + (lane >> 2);
  const int chunk = lane & 3;
  const int64_t i = r0 + row;
  const int shift = i < m ? sa[i] : 0;
  const double* mine = tile + row * kConvAPitch + chunk * 16;
  const size_t plane_stride = (size_t)m_pad * k_pad;
  int8_t* dst = planes + (size_t)(i / kBlkRows) * kBlkRows * k_pad + (size_t)kb * (kBlkRows * kBlkK) +
                (i % kBlkRows) * kBlkK + chunk * 16;
  if constexpr (KIND == 2) {
    store_bounds(mine, shift, dst);
    return;
  }
  constexpr bool TWO_LEVEL = (KIND & 1) != 0;
  Oz2SplitPair<TWO_LEVEL> xs[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) xs[u] = oz2_split_pair<TWO_LEVEL>(mine[2 * u], mine[2 * u + 1], shift);
  for (int t = 0; t < cc.N; ++t) {
    const Oz2ConvMod mod = cc.mod[t];
    unsigned v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = oz2_pack_pairs(conversion_residues<KIND>(xs[2 * u], mod), conversion_residues<KIND>(xs[2 * u + 1], mod));
    // written once, read by a later kernel: non-temporal store
    __builtin_nontemporal_store(v4u{v[0], v[1], v[2], v[3]}, reinterpret_cast<v4u*>(dst + (size_t)t * plane_stride));
  }
}

// B (k x n column-major) -> planes (row index of a plane = column j of B).  Block: 16 columns x 256 rows
// of B.  Each column segment is read coalesced (one double per lane), transposed through LDS so that a
// thread holds 16 consecutive inner-dimension values of one column, and wave w writes, for every plane,
// the 1 KiB that 16 columns x 64 bytes occupy contiguously in the output block of k-tile w.
constexpr int kConvBCols = 16;
constexpr int kConvBKC = 256;
constexpr int kConvBGroup = 18;     // doubles per 16-element group in LDS (144 bytes)
constexpr int kConvBColPitch = 296; // doubles per column in LDS: 16 groups + 8 (2368 bytes = 64 mod 256)
template <int KIND>
__device__ __forceinline__ void convert_contig(const double* __restrict__ B, int64_t ldb, int64_t k, int64_t n,
                                               int64_t n_pad, int64_t k_pad, const int* __restrict__ sb,
                                               int8_t* __restrict__ planes, const int tri, const bool cached,
                                               const Oz2ConvConsts& cc, double* tile, unsigned bx, unsigned by) {
  const int64_t j0 = (int64_t)bx * kConvBCols;  // < n_pad, multiple of 16
  const int64_t lbase = (int64_t)by * kConvBKC;
  if (KIND != 2 && !tile_used(j0, lbase, lbase + kConvBKC, (tri & 3) == 2, tri)) return;
  {
    const int64_t l = lbase + threadIdx.x;
    const int slot = (threadIdx.x >> 4) * kConvBGroup + (threadIdx.x & 15);
    auto read = [&](auto load) {
#pragma unroll 4
      for (int c = 0; c < kConvBCols; ++c) {
        const int64_t j = j0 + c;
        double v = (j < n && l < k) ? tri_value(load(B + l + j * ldb), l, j, tri) : 0.0;
        tile[c * kConvBColPitch + slot] = v;
      }
    };
    if (cached)
      read([](const double* p) { return *p; });
    else
      read([](const double* p) { return __builtin_nontemporal_load(p); });
  }
  __syncthreads();
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t l0 = lbase + wv * kBlkK + (lane & 3) * 16;
  if (lbase + wv * kBlkK >= k_pad) return;
  const int c = lane >> 2;
  const int64_t j = j0 + c;
  const int shift = j < n ? sb[j] : 0;
  const double* mine = tile + c * kConvBColPitch + (wv * 4 + (lane & 3)) * kConvBGroup;
  const size_t plane_stride = (size_t)n_pad * k_pad;
  int8_t* dst = planes + (size_t)(j / kBlkRows) * kBlkRows * k_pad + (size_t)(l0 / kBlkK) * (kBlkRows * kBlkK) +
                (j % kBlkRows) * kBlkK + (l0 % kBlkK);
  if constexpr (KIND == 2) {
    store_bounds(mine, shift, dst);
    return;
  }
  constexpr bool TWO_LEVEL = (KIND & 1) != 0;
  Oz2SplitPair<TWO_LEVEL> xs[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) xs[u] = oz2_split_pair<TWO_LEVEL>(mine[2 * u], mine[2 * u + 1], shift);
  for (int t = 0; t < cc.N; ++t) {
    const Oz2ConvMod mod = cc.mod[t];
    unsigned v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = oz2_pack_pairs(conversion_residues<KIND>(xs[2 * u], mod), conversion_residues<KIND>(xs[2 * u + 1], mod));
    // written once, read by a later kernel: non-temporal store
    __builtin_nontemporal_store(v4u{v[0], v[1], v[2], v[3]}, reinterpret_cast<v4u*>(dst + (size_t)t * plane_stride));
  }
}

// Both operands of a call in one launch (see operand_max_kernel).  KA / KB: what is written for the first /
// second job (0, 1: residue planes with the one- / two-level split; 2: the bound plane).
// FP64 operands that the last-level cache (256 MB) still holds when they are read a second time, nothing written in between: 190 MB.
// (Residue planes have their own lines, with what lies beside them there: OZ2_CACHED_RESULT those of a result, which stage 3 reads while it
// writes C; oz2_planes_through_caches those of the operands, which the products read.)
constexpr int64_t kCachedElements = (int64_t)190 << 17;
struct ConvJob {
  const double* X;
  int64_t ld, nvec, k, nvec_pad, k_pad;
  const int* shifts;
  int8_t* planes;
  int tri, strided;
  int cached;  // 1: the operands are of the last-level cache's size, which still holds them from the pass for the maxima
  unsigned gx, nblk;
};
constexpr int kConvTileDoubles =
    kConvARows * kConvAPitch > kConvBCols * kConvBColPitch ? kConvARows * kConvAPitch : kConvBCols * kConvBColPitch;
template <int KA, int KB>
__global__ void __launch_bounds__(kThreads) operand_convert_kernel(const ConvJob ja, const ConvJob jb,
                                                                   const Oz2ConvConsts cc, const Oz2ScanFinish fin) {
  __shared__ __attribute__((aligned(16))) double tile[kConvTileDoubles];
  if (fin.slots != nullptr && blockIdx.x == 0) finish_scan(fin);  // uniform over the workgroup
  if (blockIdx.x < ja.nblk) {
    const unsigned bx = blockIdx.x % ja.gx, by = blockIdx.x / ja.gx;
    if (ja.strided)
      convert_strided<KA>(ja.X, ja.ld, ja.nvec, ja.k, ja.nvec_pad, ja.k_pad, ja.shifts, ja.planes, ja.tri, ja.cached, cc, tile, bx, by);
    else
      convert_contig<KA>(ja.X, ja.ld, ja.k, ja.nvec, ja.nvec_pad, ja.k_pad, ja.shifts, ja.planes, ja.tri, ja.cached, cc, tile, bx, by);
  } else {
    const unsigned id = blockIdx.x - ja.nblk;
    const unsigned bx = id % jb.gx, by = id / jb.gx;
    if (jb.strided)
      convert_strided<KB>(jb.X, jb.ld, jb.nvec, jb.k, jb.nvec_pad, jb.k_pad, jb.shifts, jb.planes, jb.tri, jb.cached, cc, tile, bx, by);
    else
      convert_contig<KB>(jb.X, jb.ld, jb.k, jb.nvec, jb.nvec_pad, jb.k_pad, jb.shifts, jb.planes, jb.tri, jb.cached, cc, tile, bx, by);
  }
}

// ---- Vectors that fit into LDS: lines 1-5 in ONE pass, in every shift mode (in the INT8-product mode: maxima and bound planes).
// A workgroup holds eight, four or two whole vectors in LDS, so the operand is read once instead of twice and the maxima, the norms of
// the Cauchy-Schwarz mode, the shifts and the residues of both operands take one launch.  Bound by HBM at large sizes (8 bytes read, N
// written per element), by the launch and the chain of a thread's elements at small ones.  How many vectors, where not, and both sides'
// times: short_vectors.  A thread's loads are in flight together and its maximum is formed on the way; up to four k-tiles several
// waves share one, each with some of the moduli (against loads behind a branch each, eight vectors and a k-tile per wave, whole calls, us:
// 14 moduli 256^3 15.3 / 14.0, 512^3 22.7 / 21.2, 700^3 31.5 / 29.9, 1024^3 43.2 / 39.9, 13 moduli 80 x 4000 x 700 36.4 / 35.1, 16 moduli
// 150 x 2500 x 900 45.3 / 41.2; with the changes to stage 3 that came along).
// A few vectors of a column-major operand read by rows are 16- to 64-byte pieces of its columns: the workgroups of neighbouring
// groups, which read the other parts of the same cache lines, are placed on the same die.
constexpr int kShortThreads = 512;
constexpr int kShortLds = 156 * 1024;  // of 160 KiB, what a workgroup's vectors may take
constexpr int short_longest(int vectors) { return (kShortLds / (8 * vectors) - 4) / kBlkK * kBlkK; }  // padded inner dimension
static_assert(short_longest(8) == 2432 && short_longest(4) == 4928 && short_longest(2) == 9920, "the lines of short_vectors");
struct ShortJob {
  const double* X;
  int64_t ld, nvec, nvec_pad, k, k_pad;
  unsigned long long* vmax;
  unsigned long long* vnorm;  // norm bounds (mode 1), which are the reports too; KIND 2: cleared
  int* shifts;
  int8_t* planes;
  int param;  // as in ShiftJob
  int tri, strided;
  unsigned nblk;   // workgroups
  unsigned chunk;  // workgroups per die: nblk / 8, there are 256 / V or a multiple of that
};
// KIND 0, 1: residue planes as in the conversion above; 2: the plane of 6-bit bounds.  mode: as shift_of counts them (0 or 1).
// slot: this workgroup's report (mode 0; in mode 1 a vector with an infinity or a NaN has kBadReport for its norm bound)
// THROUGH: residues are stored through the caches (planes_through_caches).
template <int KIND, int V, bool THROUGH>
__device__ __forceinline__ void convert_short(const ShortJob& j, const Oz2ConvConsts& cc, const int mode, double* tile, unsigned id,
                                              unsigned long long* slot) {
  constexpr int kWaves = kShortThreads / 64;
  __shared__ unsigned long long part[kWaves][V];  // a wave's share of a vector's maximum, then of its norm
  const int64_t v0 = (int64_t)id * V;
  const int pitch = (int)j.k_pad + 4;  // doubles per vector: four banks of 32 bytes apart
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // the k-tiles that are wanted: all, or of a triangular operand's residues those that the products read (see tile_used)
  int kt_begin = 0, kt_end = (int)(j.k_pad / kBlkK);
  if (KIND != 2 && (j.tri & 3)) {
    const int64_t d0 = v0 / kBlkRows * kBlkRows;
    if (((j.tri & 3) == 1) == (j.strided != 0))
      kt_end = (int)min((int64_t)kt_end, (d0 + kBlkRows) / kBlkK);
    else
      kt_begin = (int)min((int64_t)kt_end, d0 / kBlkK);
  }
  const int begin = kt_begin * kBlkK, end = kt_end * kBlkK;
  unsigned long long mx = 0ull;
  // This thread's elements of vector v0 + v, positions l0, l0 + STEP, ...: B loads in flight at a time, none of them behind a
  // branch (beyond the operand the last element is read and zero taken).
  auto read = [&](auto batch, auto step, int v, int l0, const double* src, int64_t ld, bool swapped) {
    constexpr int B = decltype(batch)::value, STEP = decltype(step)::value;
    const bool in = v0 + v < j.nvec;
    const int last = (int)j.k - 1;
    for (int l = begin + l0; l < end; l += B * STEP) {
      double x[B];
#pragma unroll
      for (int u = 0; u < B; ++u) x[u] = src[(int64_t)min(l + u * STEP, last) * ld];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int lu = l + u * STEP;
        const double y = !in || lu > last ? 0.0 : swapped ? tri_value(x[u], lu, v0 + v, j.tri) : tri_value(x[u], v0 + v, lu, j.tri);
        if (lu < end) tile[v * pitch + lu] = y;
        const unsigned long long b = abs_bits(y);
        mx = b > mx ? b : mx;
      }
    }
  };
  auto read_all = [&](auto step, int v, int l0, const double* src, int64_t ld, bool swapped) {
    constexpr int STEP = decltype(step)::value;
    if (end - begin <= 2 * STEP)
      read(std::integral_constant<int, 2>(), step, v, l0, src, ld, swapped);
    else if (V == 8 || end - begin <= 4 * STEP)  // (V = 8: eight would cost a workgroup per compute unit)
      read(std::integral_constant<int, 4>(), step, v, l0, src, ld, swapped);
    else
      read(std::integral_constant<int, 8>(), step, v, l0, src, ld, swapped);
  };
  auto join = [&](int from, int to) {
#pragma unroll
    for (int off = from; off >= to; off >>= 1) {
      const unsigned long long o = __shfl_xor(mx, off, 64);
      mx = o > mx ? o : mx;
    }
  };
  if (j.strided) {
    const int v = threadIdx.x % V;
    read_all(std::integral_constant<int, kShortThreads / V>(), v, threadIdx.x / V, j.X + (v0 + v < j.nvec ? v0 + v : j.nvec - 1), j.ld,
             false);
    join(32, V);
    if (lane < V) part[wv][lane] = mx;
  } else {
    // kWaves / V waves take a vector, their lanes run down the vector
    const int v = wv % V;
    read_all(std::integral_constant<int, 64 * (kWaves / V)>(), v, (wv / V) * 64 + lane,
             j.X + (v0 + v < j.nvec ? v0 + v : j.nvec - 1) * j.ld, 1, true);
    join(32, 1);
    if (lane < V) part[wv][lane] = lane == v ? mx : 0ull;
  }
  __syncthreads();
  // lane: inner positions 8 (lane % 8) .. + 7 of one of the V vectors in one of the 8 / V k-tiles that a wave takes at a time;
  // wave w takes the k-tiles w, w + 8, ... (in units of kSide)
  constexpr int kSide = 8 / V;
  const int v = (lane >> 3) % V, side = lane / (8 * V);
  const int ktiles = kt_end - kt_begin, units = (ktiles + kSide - 1) / kSide;
  const double* const mine = tile + v * pitch + 8 * (lane & 7) + begin;
  mx = 0ull;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) mx = part[w][v] > mx ? part[w][v] : mx;
  unsigned long long norm = 0ull;
  if (KIND != 2 && mode == 1) {
    // (a thread's sum is exact: at most 2^11 terms of at most 2^40)
    static_assert(kShortLds / 8 / 64 <= 1 << 11, "terms of a thread");
    const int scale = mx ? 19 - exponent_of_bits(mx) : 0;
    double own = 0.0;
    for (int kt = wv * kSide + side; kt < ktiles; kt += kWaves * kSide)
#pragma unroll
      for (int u = 0; u < 8; ++u) own += scaled_ceil_sq(mine[kt * kBlkK + u], scale);
    unsigned long long sum = (unsigned long long)own;
#pragma unroll
    for (int off = 4; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
#pragma unroll
    for (int off = 32; off >= 8 * V; off >>= 1) sum += __shfl_xor(sum, off, 64);
    __syncthreads();  // the maxima have been read
    if (side == 0 && (lane & 7) == 0) part[wv][v] = sum;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) norm += part[w][v];
  }
  const int shift = shift_of(mx, norm, KIND == 2 ? 0 : mode, j.param, 0);
  if (wv == 0 && side == 0 && (lane & 7) == 0) {
    j.vmax[v0 + v] = mx;
    if (KIND == 2) j.vnorm[v0 + v] = 0ull;
    if (KIND != 2 && mode == 1) j.vnorm[v0 + v] = mx >= kInfBits ? kBadReport : norm;
    j.shifts[v0 + v] = shift;
  }
  if (wv == 0 && (KIND == 2 || mode == 0)) {
    const bool any = __any(mx >= kInfBits);
    if (lane == 0) *slot = any ? kBadReport : 0ull;
  }
  int8_t* const base = j.planes + (size_t)(v0 / kBlkRows) * kBlkRows * j.k_pad + ((v0 % kBlkRows) + v) * kBlkK + 8 * (lane & 7) +
                       (size_t)kt_begin * (kBlkRows * kBlkK);
  if constexpr (KIND == 2) {
    for (int kt = wv * kSide + side; kt < ktiles; kt += kWaves * kSide) {
      int r[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) r[u] = oz2_bound6(mine[kt * kBlkK + u], shift);
      *reinterpret_cast<v2u*>(base + (size_t)kt * (kBlkRows * kBlkK)) = v2u{pack4(r[0], r[1], r[2], r[3]), pack4(r[4], r[5], r[6], r[7])};
    }
  } else {
    // (where there are four units or less, several waves take the same one with a share of the moduli each)
    static_assert(kWaves == 8, "the shares below");
    const int parts = units > 4 ? 1 : units > 2 ? 2 : units == 2 ? 4 : 8;
    const int share = units > 4 ? 0 : units == 3 ? (wv * 11) >> 5 : units == 4 ? wv >> 2 : units == 2 ? wv >> 1 : wv;  // wv / units
    if (share >= parts) return;
    const int t0 = cc.N * share / parts, t1 = cc.N * (share + 1) / parts;
    constexpr bool TWO_LEVEL = KIND == 1;
    const size_t plane_stride = (size_t)j.nvec_pad * j.k_pad;
    for (int unit = wv - share * units; unit < units; unit += parts == 1 ? kWaves : units) {
      const int kt = unit * kSide + side;
      if (kt >= ktiles) break;
      Oz2SplitPair<TWO_LEVEL> xs[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) xs[u] = oz2_split_pair<TWO_LEVEL>(mine[kt * kBlkK + 2 * u], mine[kt * kBlkK + 2 * u + 1], shift);
      int8_t* dst = base + (size_t)t0 * plane_stride + (size_t)kt * (kBlkRows * kBlkK);
      for (int t = t0; t < t1; ++t) {
        const Oz2ConvMod mod = cc.mod[t];
        v2u w;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          w[h] = oz2_pack_pairs(oz2_residue_pair<TWO_LEVEL>(xs[2 * h], mod), oz2_residue_pair<TWO_LEVEL>(xs[2 * h + 1], mod));
        if constexpr (THROUGH)
          *reinterpret_cast<v2u*>(dst) = w;
        else
          __builtin_nontemporal_store(w, reinterpret_cast<v2u*>(dst));
        dst += plane_stride;
      }
    }
  }
}

// the flag word of the launch below, where the products are long enough to wait for it (OZ2_FINISH_FIRST_NS)
constexpr int kFinishThreads = 1024;
__global__ void __launch_bounds__(kFinishThreads) finish_scan_kernel(const Oz2ScanFinish f) { finish_scan(f); }

template <int KA, int KB, int V, bool THROUGH>
__global__ void __launch_bounds__(kShortThreads, KA == 1 || KB == 1 ? 4 : 6) short_convert_kernel(const ShortJob ja, const ShortJob jb,
                                                                      const Oz2ConvConsts cc, const int mode, const int warm,
                                                                      unsigned long long* __restrict__ slots) {
  extern __shared__ __attribute__((aligned(16))) double short_tile[];
  if (KA != 2 && warm) warm_arguments(cc);
  // workgroup i of a launch runs on die i % 8: consecutive vectors for each die; of a triangular operand, whose vectors grow from one
  // end to the other, 16 at a time, the next 16 for the next die
  const unsigned x = blockIdx.x & 7u;
  unsigned y = blockIdx.x >> 3;
  const bool first = y < ja.chunk;
  const ShortJob& j = first ? ja : jb;
  if (!first) y -= ja.chunk;
  constexpr unsigned kNear = 16 / V;  // workgroups that share the cache lines of strided vectors
  const unsigned id = j.tri ? (y / kNear * 8 + x) * kNear + y % kNear : x * j.chunk + y;
  unsigned long long* slot = slots + (first ? id : ja.nblk + id);
  if (first)
    convert_short<KA, V, THROUGH>(ja, cc, mode, short_tile, id, slot);
  else
    convert_short<KB, V, THROUGH>(jb, cc, mode, short_tile, id, slot);
}

}  // namespace

namespace {

unsigned blocks_of(int64_t v, int64_t per) { return (unsigned)((v + per - 1) / per); }

// One operand of stage 1: a set of `nvec` vectors of length k (rows of op(A) or columns of op(B)).
// strided: element (v, l) at X[v + l*ld] (vectors are rows of a column-major matrix); otherwise element
// (v, l) at X[l + v*ld] (vectors are its columns).
struct Operand {
  const double* X;
  int64_t ld;
  bool strided;
  int64_t nvec, nvec_pad, k, k_pad;
  unsigned long long* vmax;   // bit pattern of the largest magnitude per vector
  unsigned long long* vaux;   // per-vector integer norm bound, or largest element of the bound product
  unsigned long long* flag;   // set to 1 when the operand holds an infinity or a NaN
  int tri;                    // triangular structure of the stored array (see tri_value), 0 for a full matrix
  int* shifts;
  int8_t* planes;
};

// maxima of one or two operands in one launch
hipError_t launch_max(const Operand* ops, int nops, hipStream_t st) {
  MaxJob job[2] = {};
  int64_t total = 0;
  for (int x = 0; x < nops; ++x) {
    const Operand& o = ops[x];
    const int64_t gx = o.strided ? blocks_of(o.nvec, kThreads) : o.nvec;
    const int64_t gy = o.strided ? blocks_of(o.k, kRowMaxKC) : blocks_of(o.k, kColMaxKC);
    total += gx * gy;
    if (total >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    job[x] = {o.X, o.ld, o.nvec, o.k, o.vmax, o.tri, o.strided ? 1 : 0, (unsigned)gx, (unsigned)(gx * gy)};
  }
  if (nops == 1) job[1] = job[0], job[1].nblk = 0;
  hipLaunchKernelGGL(operand_max_kernel, dim3((unsigned)total), dim3(kThreads), 0, st, job[0], job[1], ops[0].flag);
  return hipSuccess;
}

void launch_norm(const Operand& o, hipStream_t st) {
  const dim3 thr(kThreads);
  if (o.strided)
    hipLaunchKernelGGL(rownorm_kernel, dim3(blocks_of(o.nvec, kThreads), blocks_of(o.k, kRowMaxKC)), thr, 0, st, o.X, o.ld,
                       o.nvec, o.k, o.vmax, o.vaux, o.tri);
  else
    hipLaunchKernelGGL(colnorm_kernel, dim3((unsigned)o.nvec, blocks_of(o.k, kColMaxKC)), thr, 0, st, o.X, o.ld, o.k, o.vmax,
                       o.vaux, o.tri);
}

// planes of one or two operands in one launch; kind 0 / 1: residue planes with the one- / two-level split,
// kind 2: the bound plane; large: operands that stream from memory (KIND 3 in the place of 1)
hipError_t launch_convert(const Operand* ops, int nops, const int* kind, bool large, const Oz2ConvConsts& conv,
                          const Oz2ScanFinish& fin, hipStream_t st) {
  ConvJob job[2] = {};
  int64_t total = 0, elements = 0;
  for (int x = 0; x < nops; ++x) {
    const Operand& o = ops[x];
    const int64_t gx = o.strided ? o.nvec_pad / kConvARows : o.nvec_pad / kConvBCols;
    const int64_t gy = o.strided ? o.k_pad / kBlkK : blocks_of(o.k_pad, kConvBKC);
    total += gx * gy;
    if (total >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    elements += o.tri ? o.nvec * o.k / 2 : o.nvec * o.k;
    job[x] = {o.X, o.ld, o.nvec, o.k, o.nvec_pad, o.k_pad, o.shifts, o.planes, o.tri, o.strided ? 1 : 0, 0, (unsigned)gx,
              (unsigned)(gx * gy)};
  }
  // Up to 190 MB the last-level cache still has the operands from the pass for the maxima, and non-temporal loads do not find them there
  // (whole calls, us, non-temporal / this: 16 moduli 300 x 300 x 20000 272 / 223, 14 moduli 500 x 500 x 12000 172 / 152, 2000 x 2000 x
  // 5000 371 / 360, INT8-product mode 1500 x 1500 x 3000 221 / 206, 3001 x 2777 x 3500 with 15 630 / 604; above, 4096^3 1048 / 1063).
  job[0].cached = job[1].cached = elements <= kCachedElements;
  const int ka = kind[0], kb = nops == 2 ? kind[1] : kind[0];
  if (nops == 1) job[1] = job[0], job[1].nblk = 0;
  const dim3 grid((unsigned)total), thr(kThreads);
#define OZ2_CONV(KA, KB) hipLaunchKernelGGL((operand_convert_kernel<KA, KB>), grid, thr, 0, st, job[0], job[1], conv, fin)
  if (ka == 2)
    OZ2_CONV(2, 2);
  else if (ka == 0 && kb == 0)
    OZ2_CONV(0, 0);
  else if (ka == 0 && large)
    OZ2_CONV(0, 3);
  else if (ka == 0)
    OZ2_CONV(0, 1);
  else if (kb == 0 && large)
    OZ2_CONV(3, 0);
  else if (kb == 0)
    OZ2_CONV(1, 0);
  else if (large)
    OZ2_CONV(3, 3);
  else
    OZ2_CONV(1, 1);
#undef OZ2_CONV
  return hipSuccess;
}

}  // namespace

// Vectors per workgroup of the one-pass conversion, or 0: the separate launches.  A workgroup's vectors have to fit its LDS, and
// several workgroups should share a compute unit, so that some read while others convert; strided vectors ask for whole cache lines, i.e.
// for many vectors.  Whole calls, us, two / four / eight vectors and separate launches, 14 moduli where not said: up to an inner dimension of
// 1024, four / eight: 512^3 21.2 / 22.2, 700^3 29.9 / 30.6, 16 moduli 150 x 2500 x 900 40.2 / 42.3, 1000 x 1000 x 200 37.0 / 36.3, 12
// moduli 1400 x 1400 x 1000 61.2 / 62.2, 2000 x 2000 x 100 57.3 / 54.5, 15 moduli 85 x 3412 x 643 35.3 / 31.9, 10 moduli
// 1900 x 1900 x 600 70.3 / 67.9.  Up to 2432: 12 moduli 150 x 150 x 1100 20.1 / 21.2 / 23.3, 27.1 separately, 16 moduli
// 1000 x 1000 x 1500 62.2 / 59.7 / 60.3, 73.9, 2048^3 183.7 / 181.0 / 182.6, 190.5, 8000 x 8000 x 2400 2390 / 2359 / 2383, 2406, dsyrk
// 3000 x 2000 214 / 210 / 219, 231.  Up to 4928: 2000 x 200 x 3000 with 15 77.5 / 84.9, 88.3, 3000^3 482 / 482, 512, 1500 x 1500 x 4500
// 229 / 213, 240, 16 moduli 4096^3 1169 / 1159, 1157, dtrmm of order 4096 with 2048 columns 522 / 525, 496.  Up to 9920: 300 x 300 x 5000
// with 16 64.2, 96.6, 500 x 500 x 8000 103, 139, 1000 x 1000 x 8000 208, 214, 2000 x 2000 x 8000 628, 607.  Elements split two levels
// deep, 22 moduli: 700 x 3000 x 4000 341 / 347, 345, 4096 x 4096 x 2048 892 / 889 / 882, 886.
// in_lines: strided vectors of which the separate launches' sixteen are whole cache lines (lines_of_vectors).  Where they are most and their
// elements many, pieces of two or four vectors cost more than the second reading (one pass, separate launches): 18 moduli
// 14272 x 139 x 1797 339, 311, both strided 10560 x 576 x 2368 498, 473, 17 moduli 352 x 4288 x 4224 301, 281, 16 moduli
// 1216 x 280 x 7424 177, 166; not in lines, 14273 vectors 347, 364, 14280 336, 354, 15 moduli both strided 3001 x 2777 x 3500 508, 536;
// below the lines 12000 x 2000 x 1600 797, 802, 14 moduli 512 x 512 x 8000, both strided 96, 113; half of them 14 moduli
// 8000 x 8000 x 2400 2227, 2263.  (Under the other shifts the separate launches take longer: 3001 x 2777 x 3500, INT8-product mode, 641, 655.)
// (strided: all strided vectors.)  Where two thirds of the vectors or more are contiguous and the last-level cache does not keep the
// operands between two readings, the one pass is the better one at every size that fits (first operand transposed where not said, one pass, separate launches): 16 moduli 4096^3 1024, 1049, 14 moduli 6000 x 6000 x 3000 1425, 1510, 16 moduli 8192^3 6743,
// 6905, 14 moduli 16000 x 300 x 4000 688, 803, 3000 x 3000 x 9000 1153, 1221, 11 moduli 1198 x 3865 x 7761 538, 596; 14 moduli 1000 x 6000 x
// 5000 as it is 531, 595, dsyrk 5000 x 8000 1324, 1373; half of them 2000 x 2000 x 5000 363, 360, 3000 x 3000 x 5000 682, 701; few 18 moduli
// 2752 x 656 x 6880 450, 395; smaller, as it is, 13 moduli 597 x 1865 x 5895 222, 208.
static int short_vectors(int64_t vectors, int64_t strided, int64_t in_lines, int64_t k_pad, bool two_level, int64_t cus) {
  const int64_t elements = vectors * k_pad;
  const bool contiguous = 3 * strided <= vectors && elements > (int64_t)19 << 20;
  const auto fits = [&](int v) { return k_pad <= short_longest(v); };
  if (k_pad <= 1024) return vectors <= (k_pad <= 256 ? 4 : k_pad <= 512 ? 8 : 12) * cus ? 4 : 8;
  if (two_level && elements > (int64_t)3 << 22) return 0;
  if (2 * in_lines > vectors && in_lines * k_pad > (int64_t)(fits(4) ? 19 : 9) << 20) return 0;
  if (fits(8)) return vectors <= 4 * cus ? 2 : 4;
  if (fits(4)) return elements > (int64_t)21 << 20 && !contiguous ? 0 : vectors <= 4 * cus || k_pad <= 3392 || two_level ? 2 : 4;
  return fits(2) && (vectors <= 8 * cus || contiguous) ? 2 : 0;
}

// Residue planes of the one-pass conversion stored through the caches: those that the last-level cache keeps for the products.  Not the
// ones of a small result that the L2s hold whole, which they would give back at the end of the launch while nothing else runs.  Whole
// calls, us, past the caches / through: 14 moduli 2000 x 2000 x 500 75.8 / 68.2, 3001 x 2777 x 200 107 / 99, 2048^3 172.1 / 166.5, 4000 x
// 500 x 1000 72.8 / 68.7, 12 moduli 8000 x 4000 x 300 332 / 319, dsyrk of order 5000 with 200 142 / 136, with 1024 and 16 moduli 315 / 307;
// 14 moduli 700^3 29.0 / 31.0, 1024^3 36.9 / 37.5; 302 MB 18 moduli 8192 x 8192 x 1024 1487 / 1507.
// Some 390 calls with up to 200 MB of planes and either more than 32 MB or 2^21 elements of C gain 2.6 % (geometric mean; operands that the
// last-level cache does not hold yet: 4.0).  Left out are the kinds that lose in both ways: results of one tile (14 moduli 117 x 90 x 5412 40.4 /
// 42.5; two tiles, 16 moduli 171 x 342 x 3113 40.4 / 40.1, operands elsewhere 47.6 / 43.1), up to 20 MB with less than 2^20 elements written
// (10 moduli 64 x 8852 x 160 27.1 / 28.8; 21 MB 12 moduli 106 x 9009 x 152 31.0 / 30.7), and long vectors that are more than 300 MB together with their
// planes (9 moduli 271 x 3981 x 4490 212 / 227; 297 MB 14 moduli 718 x 663 x 9180 186 / 184, operands elsewhere 201 / 186).  Single calls of the rest
// are slower still, most of them with planes of 32 to 48 MB (15 moduli 2085 x 178 x 1270 52.0 / 54.9, 13 moduli 16192 x 384 x 732 189 / 203; but
// 10 moduli 2095 x 154 x 1774 49.6 / 43.7).
bool oz2_planes_through_caches(int num_moduli, const Oz2Layout& lay, int64_t m, int64_t n, bool symmetric) {
  constexpr int64_t kMB = 1 << 20;
  const int64_t elements = (lay.m_pad + (symmetric ? 0 : lay.n_pad)) * lay.k_pad, bytes = num_moduli * elements, result = lay.m_pad * lay.n_pad;
  if (bytes > 200 * kMB || result <= (int64_t)OZ2_TILE_M * OZ2_TILE_N) return false;
  if (bytes > 32 * kMB) return lay.k_pad <= short_longest(8) || bytes + 8 * elements <= 300 * kMB;
  return result >= 1 << 21 && (bytes > 20 * kMB || (symmetric ? m * n / 2 : m * n) >= 1 << 20);
}

// What the shifts are formed from: the budgets of the operands, or (INT8-product mode) first the exponents 5 - e of the
// 6-bit bounds.  bit_split moves that many bits from the first operand to the second, which also gets the odd bit of the sum
// (bit_split == 0: the equal split; the symmetric product always uses it).
static void shift_params(const Oz2Plan& plan, int shift_mode, int bit_split, int param[2]) {
  if (shift_mode == OZ2_SHIFT_INT8_PRODUCT) {
    param[0] = param[1] = 6;
  } else if (shift_mode == OZ2_SHIFT_CAUCHY_SCHWARZ) {
    param[0] = plan.beta - bit_split;
    param[1] = bit_split == 0 ? plan.beta : plan.budget2 - param[0];
  } else {
    param[0] = plan.kappa - bit_split;
    param[1] = bit_split == 0 ? plan.kappa : plan.kappa_sum - param[0];
  }
}

// Are sixteen neighbouring vectors of this operand whole cache lines?
static bool lines_of_vectors(int strided, const double* X, int64_t ld) {
  return strided && ld % 16 == 0 && reinterpret_cast<uintptr_t>(X) % 128 == 0;
}

int oz2_one_pass_vectors(const Oz2Plan& plan, const Oz2Layout& lay, int strided_a, int strided_b, int lines_a, int lines_b, int symmetric,
                         int shift_mode, int bit_split, int64_t cus) {
  int param[2];
  shift_params(plan, shift_mode, bit_split, param);
  const int most = 75 - (shift_mode == OZ2_SHIFT_CAUCHY_SCHWARZ ? 1 : 0);
  const int64_t second = symmetric ? 0 : lay.n_pad;
  const int64_t in_lines = shift_mode != OZ2_SHIFT_MAX ? 0 : (lines_a ? lay.m_pad : 0) + (lines_b ? second : 0);
  const int64_t strided = (strided_a ? lay.m_pad : 0) + (strided_b ? second : 0);
  return short_vectors(lay.m_pad + second, strided, in_lines, lay.k_pad, param[0] > most || param[1] > most, cus);
}

// One operand of strided vectors, one of contiguous ones, more elements than the last-level cache keeps: the contiguous one in one
// pass (short_vectors), the scan and the conversion for the other alone, which folds both launches' reports.  Not where the vectors
// or the contiguous ones are few, nor with a triangular operand (whole calls, both in two passes / this, us: 14 moduli 3000 x 3000 x 5000
// 708 / 677, 6000 x 6000 x 3000 1510 / 1467, 16 moduli 8192 x 8192 x 4096 3749 / 3663, 10 moduli 2920 x 3916 x 3980 560 / 543, 16 moduli
// 4096^3 1037 / 1025; 15 moduli 1488 x 1744 x 8976 470 / 489, 10 moduli 1072 x 1040 x 9216 205 / 230, 18 moduli 2752 x 656 x 6880 392 / 402,
// dtrmm 4096 x 2048 443 / 461).  Vectors above 4928 are taken two at a time, which gains less, and strided ones that are not whole cache lines by
// sixteens cost the scan half of what it reads: not where those are more than the 2^25 elements up to which it is the better way for two
// operands (14 moduli, transposed, 4675 x 9173 x 9354 5016 / 5128, 16 moduli 5395 x 4159 x 7289 2504 / 2552, 10 moduli 5153 x 2649 x 6871 1123 /
// 1140; fewer 9 moduli 3674 x 3987 x 7080 1095 / 1069, in lines 17 moduli 5952 x 2880 x 5140 1.6 % faster).
int oz2_one_pass_operand(const Oz2Plan& plan, const Oz2Layout& lay, int strided_a, int strided_b, int lines_a, int lines_b, int triangular,
                         int symmetric, int shift_mode, int bit_split, int64_t cus) {
  int param[2];
  shift_params(plan, shift_mode, bit_split, param);
  if (symmetric || triangular || shift_mode != OZ2_SHIFT_MAX || !strided_a == !strided_b || param[0] > 75 || param[1] > 75) return 0;
  const int64_t vectors = lay.m_pad + lay.n_pad, contiguous = strided_a ? lay.n_pad : lay.m_pad;
  const bool fits = lay.k_pad > short_longest(8) && lay.k_pad <= short_longest(2);
  if (!fits || 3 * contiguous < vectors || vectors * lay.k_pad <= kCachedElements || vectors < 20 * cus) return 0;
  if (lay.k_pad > short_longest(4) && !(strided_a ? lines_a : lines_b) && (vectors - contiguous) * lay.k_pad > (int64_t)1 << 25) return 0;
  return strided_a ? 2 : 1;
}

hipError_t oz2_launch_finish_scan(const Oz2ScanFinish& f, hipStream_t st) {
  hipLaunchKernelGGL(finish_scan_kernel, dim3(1), dim3(kFinishThreads), 0, st, f);
  return hipGetLastError();
}

// Once per process, before any launch: the dynamic LDS limit of the one-pass conversion.
hipError_t oz2_stage1_setup() {
#define OZ2_ALL(KA, KB, THROUGH)                                           \
  reinterpret_cast<const void*>(short_convert_kernel<KA, KB, 8, THROUGH>), \
      reinterpret_cast<const void*>(short_convert_kernel<KA, KB, 4, THROUGH>), \
      reinterpret_cast<const void*>(short_convert_kernel<KA, KB, 2, THROUGH>)
#define OZ2_BOTH(KA, KB) OZ2_ALL(KA, KB, false), OZ2_ALL(KA, KB, true)
  const void* kernels[27] = {OZ2_BOTH(0, 0), OZ2_BOTH(0, 1), OZ2_BOTH(1, 0), OZ2_BOTH(1, 1), OZ2_ALL(2, 2, false)};
#undef OZ2_BOTH
#undef OZ2_ALL
  hipError_t e = hipSuccess;
  for (int i = 0; i < 27 && e == hipSuccess; ++i)
    e = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, kShortLds);
  return e;
}

// transa / transb: 0 = the operand is stored as op(X) (column-major), 1 = it is stored transposed.
// B == nullptr: the symmetric product op(A) op(A)^T (n == m); only A's vectors, shifts and planes are produced.
// tri_a / tri_b: triangular structure of the stored arrays (0 = full; see tri_value).
// strassen: lay is the layout of the Strassen form; shifts (and the bound product of the INT8-product mode) are
// formed as usual on its padded extents, only the residue planes differ.
hipError_t oz2_launch_stage1(int transa, int transb, int64_t m, int64_t n, int64_t k, const double* A, int64_t lda,
                             const double* B, int64_t ldb, int tri_a, int tri_b, const Oz2Plan& plan, int shift_mode,
                             int bit_split, int strassen, const Oz2Layout& lay, char* ws, hipStream_t st, int thin,
                             int* large_two_level, Oz2ScanFinish* deferred) {
  // rows of op(A): strided in a stored m x k matrix, contiguous in a stored k x m matrix;
  // columns of op(B): contiguous in a stored k x n matrix, strided in a stored n x k matrix
  // Row maxima, flag words and column maxima are adjacent, and so are the two auxiliary vectors: one fill
  // launch clears each group.
  if (lay.off_flags != lay.off_rowmax + (size_t)lay.m_pad * 8 || lay.off_colmax != lay.off_flags + 256 ||
      lay.off_colnorm != lay.off_rownorm + (size_t)lay.m_pad * 8)
    return hipErrorInvalidValue;
  unsigned long long* flag = reinterpret_cast<unsigned long long*>(ws + lay.off_flags);
  const Operand ops[2] = {
      {A, lda, transa == 0, m, lay.m_pad, k, lay.k_pad, reinterpret_cast<unsigned long long*>(ws + lay.off_rowmax),
       reinterpret_cast<unsigned long long*>(ws + lay.off_rownorm), flag, tri_a,
       reinterpret_cast<int*>(ws + lay.off_sa), reinterpret_cast<int8_t*>(ws + lay.off_a)},
      {B, ldb, transb != 0, n, lay.n_pad, k, lay.k_pad, reinterpret_cast<unsigned long long*>(ws + lay.off_colmax),
       reinterpret_cast<unsigned long long*>(ws + lay.off_colnorm), flag, tri_b,
       reinterpret_cast<int*>(ws + lay.off_sb), reinterpret_cast<int8_t*>(ws + lay.off_b)}};
  const dim3 thr(kThreads);
  const int nops = B ? 2 : 1;
  const int64_t n_max = nops == 2 ? lay.m_pad + 32 + lay.n_pad : lay.m_pad + 32;
  const int64_t n_aux = nops == 2 ? lay.m_pad + lay.n_pad : lay.m_pad;
  const Oz2ScanFinish nothing = {nullptr, 0u, nullptr, 0};
  auto fill = [&](unsigned long long* p, int64_t count) {
    hipLaunchKernelGGL(fill_u64_kernel, dim3(blocks_of(count, kThreads)), thr, 0, st, p, count);
  };
  auto shifts = [&](int mode, int param_a, int param_b, int off_a, int off_b) {
    const ShiftJob ja = {ops[0].vmax, ops[0].vaux, ops[0].shifts, ops[0].nvec_pad, param_a, off_a};
    const ShiftJob jb = {ops[1].vmax, ops[1].vaux, ops[1].shifts, nops == 2 ? ops[1].nvec_pad : 0, param_b, off_b};
    hipLaunchKernelGGL(shifts_kernel, dim3(blocks_of(ja.count + jb.count, kThreads)), thr, 0, st, ja, jb, mode);
  };
  Oz2ConvConsts conv = plan.conv;
  const int d = bit_split;
  int xbits[2];  // |x'| < 2^xbits decides how deep the conversion kernels split an element
  Oz2ScanFinish fin = nothing;
  if (deferred) *deferred = nothing;
  const int64_t vectors = lay.m_pad + (nops == 2 ? lay.n_pad : 0);
  int param[2];
  shift_params(plan, shift_mode, d, param);
  const int base_mode = shift_mode == OZ2_SHIFT_CAUCHY_SCHWARZ ? 1 : 0;  // as shift_of counts them
  // Short vectors: everything in one launch (in the INT8-product mode: maxima and bound planes), whose reports the caller's
  // GEMM launch turns into the flag word (deferred != nullptr: the caller sees to that).
  const bool two_a = param[0] + base_mode > 75, two_b = param[1] + base_mode > 75;
  const bool lines_a = lines_of_vectors(ops[0].strided, A, lda), lines_b = lines_of_vectors(ops[1].strided, B, ldb);
  const int short_vecs = deferred && !thin && !strassen ? oz2_one_pass_vectors(plan, lay, ops[0].strided, ops[1].strided, lines_a, lines_b,
                                                                               nops == 1, shift_mode, d, oz2_gemm_cus())
                                                        : 0;
  if (short_vecs) {
    ShortJob sj[2] = {};
    unsigned groups = 0;
    for (int x = 0; x < nops; ++x) {
      const Operand& o = ops[x];
      const unsigned nblk = (unsigned)(o.nvec_pad / short_vecs);
      sj[x] = {o.X, o.ld, o.nvec, o.nvec_pad, o.k, o.k_pad, o.vmax, o.vaux, o.shifts, o.planes, param[x], o.tri,
               o.strided ? 1 : 0, nblk, nblk / 8};
      groups += nblk;
    }
    // The reports live in the auxiliary vectors: a word per two vectors or more, or, in the Cauchy-Schwarz mode, whose norm bounds
    // belong there, a word per vector; in the INT8-product mode, whose auxiliary vectors are cleared for the product's maxima, in plane 1 of the
    // operand with more vectors, which the launch after the bound product writes (at least 64 bytes per vector, two moduli at least).
    const bool bounds = shift_mode == OZ2_SHIFT_INT8_PRODUCT;
    const Operand& most = ops[nops == 2 && lay.n_pad > lay.m_pad ? 1 : 0];
    unsigned long long* slots =
        bounds ? reinterpret_cast<unsigned long long*>(most.planes + (size_t)most.nvec_pad * most.k_pad) : ops[0].vaux;
    // (Inputs with an infinity or a NaN skip their products, except short ones of short vectors: there the look at the reports would
    // cost up to 6 % of a finite call, Cauchy-Schwarz mode 500^3 22.2 -> 23.5 us.)
    fin = {slots, base_mode == 1 ? (unsigned)vectors : groups, flag, lay.k_pad > 1024};
    const dim3 grid(8 * (sj[0].chunk + sj[1].chunk)), thr(kShortThreads);
    // Up to three workgroups on two compute units wait for the constants (700^3 29.8 -> 29.2 us a call), and those of vectors above 1024
    // too (300 x 300 x 1500 29.1 -> 28.2, 2048 x 256 x 2000 59.3 -> 58.0); where more have short vectors, the first have fetched them for
    // the others and the loads only cost (9 moduli 71 x 5081 x 184 22.5 -> 23.1, 900 x 700 x 300 22.7 -> 23.1).
    const int warm = lay.k_pad > 1024 || 2 * (int64_t)groups <= 3 * oz2_gemm_cus();
    const size_t lds = (size_t)short_vecs * (lay.k_pad + 4) * sizeof(double);
    const bool through = oz2_planes_through_caches(plan.N, lay, m, n, B == nullptr);
#define OZ2_SHORT_V(KA, KB, V, THROUGH) \
  hipLaunchKernelGGL((short_convert_kernel<KA, KB, V, THROUGH>), grid, thr, lds, st, sj[0], sj[1], conv, base_mode, warm, slots)
#define OZ2_SHORT_ALL(KA, KB, THROUGH)    \
  do {                                    \
    if (short_vecs == 8)                  \
      OZ2_SHORT_V(KA, KB, 8, THROUGH);    \
    else if (short_vecs == 4)             \
      OZ2_SHORT_V(KA, KB, 4, THROUGH);    \
    else                                  \
      OZ2_SHORT_V(KA, KB, 2, THROUGH);    \
  } while (0)
#define OZ2_SHORT(KA, KB)                 \
  do {                                    \
    if (through)                          \
      OZ2_SHORT_ALL(KA, KB, true);        \
    else                                  \
      OZ2_SHORT_ALL(KA, KB, false);       \
  } while (0)
    if (bounds)
      OZ2_SHORT_ALL(2, 2, false);
    else if (two_a && two_b)
      OZ2_SHORT(1, 1);
    else if (two_a)
      OZ2_SHORT(1, 0);
    else if (two_b)
      OZ2_SHORT(0, 1);
    else
      OZ2_SHORT(0, 0);
#undef OZ2_SHORT
#undef OZ2_SHORT_ALL
#undef OZ2_SHORT_V
    if (!bounds) {
      *deferred = fin;
      return hipGetLastError();
    }
  }
  // Small operands: maxima, norm bounds and shifts in one launch without atomics (nothing to clear
  // first); its per-workgroup reports become the flag word in the conversion launch.  "Small": at most 2^25 elements
  // in both operands together (4096 x 4096 twice), where 16 vectors per workgroup are work enough for the chip
  // and the launches saved still count.  In the modes of Section 4.1 few long vectors keep the separate launches, which give a
  // vector several workgroups: where their number is below an eighth (mode 2 with two operands: a tenth) of their length, and that
  // above a line, the scan's workgroups are too few and too long (whole calls, 14 moduli, scan / separate launches, us, plain
  // operands and with the first one transposed: mode 1 256 x 256 x 8192 103 / 102 and 85 / 99, x 12000 151 / 125 and 134 / 119,
  // x 32768 378 / 265 and 344 / 253, 64 x 64 x 10300 130 / 119 and 105 / 114, 500 x 500 x 16384 293 / 254, 1000 x 1000 x 8192
  // 252 / 258, x 16384 500 / 469 and 432 / 442; mode 2 256 x 256 x 4096 131 / 144 and 121 / 139, x 10300 246 / 231 and 230 / 226,
  // 500 x 500 x 10300 315 / 298 and 295 / 296, 1000 x 1000 x 16384 692 / 696 and 659 / 678; dsyrk, mode 1 order 500, 8192
  // 138 / 121 and 109 / 116, 10000 169 / 141 and 144 / 130, order 900, 10000 218 / 194, mode 2 order 500, 10000 277 / 260 and
  // 254 / 253, order 900, 12000 384 / 358).
  const int line = nops == 1 ? 8192 : shift_mode == OZ2_SHIFT_CAUCHY_SCHWARZ ? 12288 : 10240;
  const int64_t few = lay.k_pad / (nops == 2 && shift_mode == OZ2_SHIFT_INT8_PRODUCT ? 10 : 8);
  const bool few_and_long = shift_mode != OZ2_SHIFT_MAX && lay.k_pad > line && vectors <= few;
  const bool large = vectors * lay.k_pad > ((int64_t)1 << 25);
  const bool scan = !strassen && !large && !few_and_long;
  const int alone = !strassen && !thin && !short_vecs
                        ? oz2_one_pass_operand(plan, lay, ops[0].strided, ops[1].strided, lines_a, lines_b, tri_a || tri_b, nops == 1, shift_mode, d,
                                               oz2_gemm_cus())
                        : 0;
  if (short_vecs) {
    // (the bound planes exist)
  } else if (alone) {
    const Operand &c = ops[alone - 1], &o = ops[2 - alone];
    const int v = lay.k_pad > short_longest(4) || lay.k_pad <= 3392 || c.nvec_pad <= 4 * oz2_gemm_cus() ? 2 : 4;
    const unsigned nblk = (unsigned)(c.nvec_pad / v), scans = (unsigned)(o.nvec_pad / kScanVecs);
    unsigned long long* slots = reinterpret_cast<unsigned long long*>(ws + lay.off_c);
    const ShortJob sj = {c.X, c.ld, c.nvec, c.nvec_pad, c.k, c.k_pad, c.vmax, c.vaux, c.shifts, c.planes, param[alone - 1], 0, 0, nblk, nblk / 8};
    ShortJob none = sj;
    none.nblk = none.chunk = 0;
    const size_t lds = (size_t)v * (lay.k_pad + 4) * sizeof(double);
    if (v == 2)
      hipLaunchKernelGGL((short_convert_kernel<0, 0, 2, false>), dim3(8 * sj.chunk), dim3(kShortThreads), lds, st, sj, none, conv, 0, 1, slots);
    else
      hipLaunchKernelGGL((short_convert_kernel<0, 0, 4, false>), dim3(8 * sj.chunk), dim3(kShortThreads), lds, st, sj, none, conv, 0, 1, slots);
    const ScanJob job = {o.X, o.ld, o.nvec, o.nvec_pad, o.k, o.vmax, o.vaux, o.shifts, param[2 - alone], o.tri, o.strided ? 1 : 0, scans};
    ScanJob no_job = job;
    no_job.nblk = 0;
    hipLaunchKernelGGL(vector_scan_kernel, dim3(scans), dim3(kScanThreads), 0, st, job, no_job, 0, slots + nblk);
    fin = {slots, nblk + scans, flag, 0};
    const int kind[1] = {0};
    if (hipError_t e = launch_convert(&o, 1, kind, false, conv, fin, st); e != hipSuccess) return e;
    return hipGetLastError();
  } else if (scan) {
    ScanJob sj[2] = {};
    unsigned total = 0;
    for (int x = 0; x < nops; ++x) {
      const Operand& o = ops[x];
      sj[x] = {o.X, o.ld, o.nvec, o.nvec_pad, o.k, o.vmax, o.vaux, o.shifts, param[x], o.tri, o.strided ? 1 : 0,
               (unsigned)(o.nvec_pad / kScanVecs)};
      total += sj[x].nblk;
    }
    if (nops == 1) sj[1] = sj[0], sj[1].nblk = 0;
    // the slots live in the product region, which nothing else uses before the products (one word per 16 vectors)
    unsigned long long* slots = reinterpret_cast<unsigned long long*>(ws + lay.off_c);
    hipLaunchKernelGGL(vector_scan_kernel, dim3(total), dim3(kScanThreads), 0, st, sj[0], sj[1], base_mode, slots);
    fin = {slots, total, flag, 0};
  } else {
    fill(ops[0].vmax, n_max);
    if (hipError_t e = launch_max(ops, nops, st); e != hipSuccess) return e;
    if (base_mode == 1) {
      fill(ops[0].vaux, n_aux);
      for (int x = 0; x < nops; ++x) launch_norm(ops[x], st);
    }
    shifts(base_mode, param[0], param[1], 0, 0);
  }
  if (shift_mode == OZ2_SHIFT_INT8_PRODUCT) {
    // bound planes (in the slots of residue plane 0), their INT8 product (in the slot of product plane 0),
    // its row and column maxima, then the shifts.  In the symmetric case the product is A''A''^T and its
    // row maxima are its column maxima (those land in the unused column array).
    if (!short_vecs) {
      const int bound[2] = {2, 2};
      if (hipError_t e = launch_convert(ops, nops, bound, false, conv, fin, st); e != hipSuccess) return e;
      fin = nothing;
      if (!scan) fill(ops[0].vaux, n_aux);
    }
    const int tile = oz2_bound_tile(lay, m, n, B == nullptr, oz2_gemm_cus());
    if (tile != 256) {
      if (hipError_t e = oz2_launch_bound_maxima(tile, lay, ws, m, n, B == nullptr, fin, st); e != hipSuccess) return e;
      fin = nothing;
    } else {
      if (fin.slots)
        if (hipError_t e = oz2_launch_finish_scan(fin, st); e != hipSuccess) return e;
      fin = nothing;
      if (hipError_t e = oz2_launch_bound_gemm(lay, ws, B == nullptr, st); e != hipSuccess) return e;
      const int64_t row_blocks = (lay.m_pad + kProdRows - 1) / kProdRows;
      int cols = 8;  // as few as leave a row 128 atomic maxima or fewer
      while (cols < 64 && (n + cols - 1) / cols > 128) cols *= 2;
      const int64_t nblk = row_blocks * (int64_t)blocks_of(n, cols);
      if (nblk >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
      hipLaunchKernelGGL(prodmax_kernel, dim3((unsigned)nblk), thr, 0, st, reinterpret_cast<const int*>(ws + lay.off_c),
                         lay.m_pad, m, n, row_blocks, cols, ops[0].vaux, ops[1].vaux);
    }
    shifts(2, plan.budget2, plan.budget2, -d, d);
    xbits[0] = plan.budget2 / 2 + 7 - d;  // |x'| < 2^(e + 1 + sa) <= 2^(floor(b/2) + 6 -+ d)
    xbits[1] = plan.budget2 / 2 + 7 + d;
  } else {
    xbits[0] = param[0] + base_mode;
    xbits[1] = param[1] + base_mode;
  }
  const int kinds[2] = {xbits[0] > 75 ? 1 : 0, xbits[1] > 75 ? 1 : 0};
  if (strassen) {
    // general products only: the planes are the seven block combinations per modulus of the Strassen form
    if (!B || tri_a || tri_b) return hipErrorInvalidValue;
    return oz2_launch_strassen_convert(transa, transb, m, n, k, A, lda, B, ldb, plan, kinds, lay, ws, st);
  }
  if (thin) {
    const int small = thin == 1 ? 1 : 0;
    *large_two_level = kinds[1 - small];
    if (hipError_t e = launch_convert(ops + small, 1, kinds + small, large, conv, fin, st); e != hipSuccess) return e;
    return hipGetLastError();
  }
  if (hipError_t e = launch_convert(ops, nops, kinds, large, conv, fin, st); e != hipSuccess) return e;
  return hipGetLastError();
}

template <bool TWO_LEVEL>
static bool host_residues(const Oz2ConvConsts& c, double a, int shift, int8_t* out) {
  const Oz2SplitPair<TWO_LEVEL> s = oz2_split_pair<TWO_LEVEL>(a, a, shift);
  bool same = true;
  for (int t = 0; t < c.N; ++t) {
    const oz2_u16x2 r = oz2_residue_pair<TWO_LEVEL>(s, c.mod[t]);
    out[t] = (int8_t)(oz2_pack_pairs(r, r) & 0xff);
    if constexpr (TWO_LEVEL) {
      const oz2_u16x2 l = oz2_residue_pair_lean<true>(s, c.mod[t]), m = oz2_residue_pair_lean<false>(s, c.mod[t]);
      same = same && l[0] == r[0] && l[1] == r[1] && m[0] == r[0] && m[1] == r[1];
    }
  }
  return same;
}
bool oz2_host_residues_impl(const Oz2ConvConsts& c, double a, int shift, int8_t* out) {
  return c.two_level ? host_residues<true>(c, a, shift, out) : host_residues<false>(c, a, shift, out);
}
