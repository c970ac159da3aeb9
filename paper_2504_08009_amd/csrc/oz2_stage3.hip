// Stages 3 and 4 of Ozaki scheme II on gfx950: Algorithm 1 lines 7-11 fused in one pass.
//   per output element: c''_t = c'_t mod p_t (line 7), Y = sum_t c''_t W_t on 40-bit FP64 limbs (line 9),
//   X = Y mod M in the symmetric range (line 10), one rounding to FP64 and the exact power-of-two
//   scaling by 2^-(sa_i + sb_j) (line 11).
// 4N (INT32 planes) or N (UINT8 residue planes, line 7 already taken by the GEMM epilogue) bytes read and 8
// written per element: bound by HBM traffic with INT32 planes, by FP64 instruction issue with UINT8 planes.
#include "oz2_fallback_tile.h"
#include "oz2_fast_div.h"
#include "oz2_math.h"
#include "oz2_route.h"
#include "oz2_warm.h"

namespace {

constexpr int kThreads = 256;
static_assert(kThreads == kFallbackThreads, "the small-problem kernel runs both bodies with one block size");

// Two elements of C, past the caches: what this launch writes is not read by it again, and left in the L2s it would be given back at the
// end of the launch, while nothing else runs (whole calls, us, through / past: 14 moduli 2048^3 177.3 / 169.2, 1000 x 1000 x 300 31.2 /
// 29.3, 1024^3 37.9 / 37.3, 12 moduli dsyrk of order 5000 with 200 139.5 / 135.8, 18 moduli 8192 x 8192 x 1024 1502 / 1483; dtrmm 9024 x 1696 2.6 %
// faster, 3000^3 1.5 %, but 6000 x 2500 1.7 % slower, 4096 x 2048 0.7 %).
__device__ __forceinline__ void store_past(double* dst, double lo, double hi) {
  typedef double v2d __attribute__((ext_vector_type(2)));
  __builtin_nontemporal_store(v2d{lo, hi}, reinterpret_cast<v2d*>(dst));
}

// One plane's values for R consecutive rows: INT32 products (16-byte loads, R = 4) or UINT8 residues that
// the GEMM epilogue already reduced (R bytes: 4 or 2).
template <bool U8, int R>
struct PlaneLoad;
template <>
struct PlaneLoad<false, 4> {
  typedef int Raw __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ void residues(const Raw& c, double p, double ip, double hip_, double* res) {
    res[0] = oz2_floor_mod(c.x, p, ip, hip_);
    res[1] = oz2_floor_mod(c.y, p, ip, hip_);
    res[2] = oz2_floor_mod(c.z, p, ip, hip_);
    res[3] = oz2_floor_mod(c.w, p, ip, hip_);
  }
};
template <>
struct PlaneLoad<true, 4> {
  typedef unsigned Raw;
  static __device__ __forceinline__ void residues(Raw c, double, double, double, double* res) {
#pragma unroll
    for (int r = 0; r < 4; ++r) res[r] = (double)((c >> (8 * r)) & 0xffu);
  }
};
template <>
struct PlaneLoad<true, 2> {
  typedef unsigned short Raw;
  static __device__ __forceinline__ void residues(Raw c, double, double, double, double* res) {
    res[0] = (double)(c & 0xffu);
    res[1] = (double)(c >> 8);
  }
};

// One thread: the R consecutive rows i0 .. of one column j.  kBatch planes' values are fetched at a time, one batch ahead of
// the arithmetic.  SMALL (a launch at its own latency): the shifts and C, where it is updated, are fetched with the first ones,
// and so is *flag, which leaves C alone where it is set: one wait for memory in the place of four (256^3, inside the launch, 3.3
// us before; in large launches the registers cost a wave per SIMD).
// PASS_BY: planes larger than the last-level cache are read past the caches; smaller ones are found there.
template <int L, bool U8, int R, int kBatch, bool SMALL, bool PASS_BY>
__device__ __forceinline__ void crt_rows(const void* __restrict__ cplanes, int64_t m_pad, int64_t n_pad,
                                         const int* __restrict__ sa, const int* __restrict__ sb, double* __restrict__ C,
                                         int64_t ldc, int64_t m, int64_t n, const double alpha, const double beta,
                                         const int triangle, const Oz2CrtConsts& cc, const int64_t j, const int64_t i0,
                                         const unsigned long long* __restrict__ flag) {
  typedef PlaneLoad<U8, R> PL;
  typedef typename PL::Raw Raw;
  // symmetric product: only the lower (1: i >= j) or upper (2: i <= j) triangle of C exists and is written
  if ((triangle == 1 && i0 + R - 1 < j) || (triangle == 2 && i0 > j)) return;
  // element (i, j) of plane t sits at index (t*n_pad + j)*m_pad + i, in units of int32 or of bytes
  const size_t elem = (size_t)j * m_pad + i0;
  const Raw* src = reinterpret_cast<const Raw*>(static_cast<const char*>(cplanes) + elem * (U8 ? 1 : 4));
  const size_t stride = (size_t)n_pad * m_pad * (U8 ? 1 : 4) / sizeof(Raw);

  double S[R][L];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int l = 0; l < L; ++l) S[r][l] = 0.0;

  // Planes are read once, a batch ahead of the arithmetic: kBatch loads per thread in flight keep enough bytes
  // moving per CU to cover the memory latency (one load ahead does not).
  const int N = cc.N;
  Raw nxt[kBatch];
  auto read = [](const Raw* p) { return PASS_BY ? __builtin_nontemporal_load(p) : *p; };
#pragma unroll
  for (int d = 0; d < kBatch; ++d) nxt[d] = read(src + (size_t)(d < N ? d : N - 1) * stride);
  double* dst = C + i0 + j * ldc;
  int shift[R];
  double old[R];
  auto mine = [&](int r) { return i0 + r < m && !(triangle == 1 && i0 + r < j) && !(triangle == 2 && i0 + r > j); };
  if constexpr (SMALL) {
    const int sbj = sb[j];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      shift[r] = sa[i0 + r] + sbj;
      old[r] = beta == 0.0 || !mine(r) ? 0.0 : dst[r];
    }
    if (*flag != 0ull) return;
  }
  for (int t0 = 0; t0 < N; t0 += kBatch) {
    Raw cur[kBatch];
#pragma unroll
    for (int d = 0; d < kBatch; ++d) cur[d] = nxt[d];
    if (t0 + kBatch < N) {
#pragma unroll
      for (int d = 0; d < kBatch; ++d) {
        const int t = t0 + kBatch + d;
        nxt[d] = read(src + (size_t)(t < N ? t : N - 1) * stride);  // past the end: a harmless repeat of the last plane
      }
    }
#pragma unroll
    for (int d = 0; d < kBatch; ++d) {
      const int t = t0 + d;
      if (t < N) {
        double res[R];
        PL::residues(cur[d], cc.p[t], cc.inv_p[t], cc.half_inv_p[t], res);
#pragma unroll
        for (int l = 0; l < L; ++l) {
          const double w = cc.w[t][l];
#pragma unroll
          for (int r = 0; r < R; ++r) S[r][l] = fma(res[r], w, S[r][l]);
        }
      }
    }
  }
  const int sbj = SMALL ? 0 : sb[j];
  double out[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int e2;
    const double x = oz2_crt_reduce<L>(S[r], cc, &e2);
    if constexpr (SMALL)
      out[r] = ldexp(x, e2 - shift[r]);
    else
      out[r] = ldexp(x, e2 - sa[i0 + r] - sbj);  // sa is padded to m_pad (a multiple of 256): readable
  }
  if (alpha != 1.0 || beta != 0.0) {
    // C := alpha * P + beta * C with one rounding of beta * C and one fused multiply-add; C is not read when
    // beta is zero (BLAS convention)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double c = SMALL ? old[r] : (beta == 0.0 || !mine(r)) ? 0.0 : dst[r];
      out[r] = fma(alpha, out[r], beta == 0.0 ? 0.0 : beta * c);
    }
  }
  // all R results of the thread leave together: its 8 R contiguous bytes complete their cache lines at once
  const bool whole = triangle == 0 || (triangle == 1 && i0 >= j) || (triangle == 2 && i0 + R - 1 <= j);
  if (whole && i0 + R <= m && ((reinterpret_cast<uintptr_t>(dst) & 15) == 0)) {
#pragma unroll
    for (int r = 0; r < R; r += 2) {
      if constexpr (R == 2)  // the smallest results, a launch at its own latency: through the caches (14 moduli 323 x 1437 26.1, past 26.6)
        *reinterpret_cast<double2*>(dst + r) = make_double2(out[r], out[r + 1]);
      else
        store_past(dst + r, out[r], out[r + 1]);
    }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (i0 + r < m && !(triangle == 1 && i0 + r < j) && !(triangle == 2 && i0 + r > j)) dst[r] = out[r];
  }
}

// The work of a launch is the columns' pieces of R rows, one after the other (per_col of them in a column), so that
// short and ragged columns leave no lanes idle (a block per 2048 rows of a column before: one lane in eight worked at 256
// rows, two thirds of them at 2777).  A launch takes the columns j0 .. n - 1.
template <int L, bool U8, int R, bool PASS_BY>
__global__ void __launch_bounds__(kThreads) crt_kernel(const void* __restrict__ cplanes, int64_t m_pad, int64_t n_pad,
                                                       const int* __restrict__ sa, const int* __restrict__ sb,
                                                       double* __restrict__ C, int64_t ldc, int64_t m, int64_t j0,
                                                       int64_t n, const double alpha, const double beta,
                                                       const unsigned long long* __restrict__ skip_flag,
                                                       const int triangle, const int per_col, const FastDiv by_col,
                                                       const Oz2CrtConsts cc) {
  // a non-finite input was found in stage 1: C is left to the FP64 fallback (uniform over the grid)
  if (skip_flag != nullptr && *skip_flag != 0ull) return;
  const int g = (int)(blockIdx.x * kThreads + threadIdx.x), q = g / by_col;
  const int64_t j = j0 + q;
  if (j >= n) return;
  crt_rows<L, U8, R, 4, false, PASS_BY>(cplanes, m_pad, n_pad, sa, sb, C, ldc, m, n, alpha, beta, triangle, cc, j, (int64_t)(g - q * per_col) * R,
                        nullptr);
}

// Products below 2^24 elements, where every launch counts: the blocks of the FP64 fallback ride in the same launch, behind those of
// the kernel above.  Which of the two sets works is decided by the flag of stage 1, the other returns at once.
// kBatch: eight planes at a time, four where the last eight would be half repeats of the last plane or more (9 to 12 moduli, say), which
// are fetched like any other (whole calls, us, always eight / this: 4 moduli 1629 x 3786 x 343 57.9 / 56.0, 10 moduli 2000 x 2000 x 300
// 58.7 / 57.5, 9 moduli 2500 x 2500 x 200 with an update 80.3 / 79.1; always four / this: 15 moduli 3001 x 2777 x 300 131.6 / 129.4, 14 moduli 700^3 29.7 / 29.4).
template <int L, int R, int kBatch, bool PASS_BY>
__global__ void __launch_bounds__(kThreads, 4) crt_or_fallback_kernel(const void* __restrict__ cplanes, int64_t m_pad,
                                                                   int64_t n_pad, const int* __restrict__ sa,
                                                                   const int* __restrict__ sb,
                                                                   const unsigned long long* __restrict__ flag,
                                                                   const unsigned crt_blocks, const int per_col,
                                                                   const FastDiv by_col, const Oz2FallbackArgs f,
                                                                   const Oz2CrtConsts cc) {
  warm_arguments(cc);
  if (blockIdx.x < crt_blocks) {
    const int g = (int)(blockIdx.x * kThreads + threadIdx.x), j = g / by_col;
    if (j >= f.n) return;
    crt_rows<L, true, R, kBatch, true, PASS_BY>(cplanes, m_pad, n_pad, sa, sb, f.C, f.ldc, f.m, f.n, f.alpha, f.beta, 0, cc, j,
                            (int64_t)(g - j * per_col) * R, flag);
  } else if (*flag != 0ull) {
    oz2_fallback_tile<kFallbackSmallTile>(f, blockIdx.x - crt_blocks);
  }
}

// ---------------------------------------------------------------------------------------------------
// Lines 8-11 on UINT8 residue planes with the accumulation of line 9 on the matrix cores (at most OZ2_MFMA_N moduli).
// Y = sum_t c''_t W_t is a product of the residues (elements x moduli, bytes) with the weights (moduli x digits,
// bytes once the weights are written in balanced base-256 digits): one v_mfma_i32_32x32x32_i8 forms all sixteen
// digit sums of 64 output elements.  Operand roles: the 32 "rows" of the first operand run over the result
// registers and hold the digits, rows 0-15 with their weights on inner positions 0-15 and rows 16-31 with the same
// weights on inner positions 16-31; a lane of the second operand supplies inner positions 16 (lane / 32) + 0..15 of
// column lane % 32, i.e. the sixteen residues of ITS OWN element.  Lanes 0-31 therefore multiply against rows 0-15,
// lanes 32-63 against rows 16-31, and every lane's element gets its sixteen digit sums, half of them in the lane
// itself and half in the lane 32 away (result register e of lane l is row 8 (e / 4) + 4 (l / 32) + e % 4); eight
// v_permlane32_swap bring them together.  The residues enter as c'' - 128 (signed bytes); 128 sum_t dig, in limb
// form, is added when the digits become the 40-bit limbs the exact tail works on.
// WIDE, 17 to 20 moduli: twenty digits, on the rows of ten result registers of both halves (digit e or 10 + e), and two products, one for
// the elements of lanes 0-31 and one for those of lanes 32-63, whose twenty residues are shared out between the halves: words 0 and 1 in
// the lower one, 3 and 4 in the upper, brought there by two v_permlane32_swap for both products; word 2 stays where it is, against weights
// that are zero in the other half.  (Four products, two more for digits 16-19 of either half, took 135 registers and were slower than
// crt_kernel: 660 against 480 us for 18 moduli at 8192 x 8192; with products of 32 x 32 x 16, whose constants take fewer registers, 15 us
// slower than this there.)  Whole calls, us, crt_kernel / this: 18 moduli 8192 x 8192 x 1024 1565 / 1505, x 200 1032 / 968, 20 moduli x 200
// 1101 / 1050, 17 moduli 5000 x 7999 x 300 with an update 771 / 698.
// A thread owns four consecutive rows (one 32-bit load per plane, transposed to four 16-byte operands with byte
// permutes) of kCrtCols consecutive columns, so that the set-up of the constant operand is spread over 64 elements.
// Residues, and C where it is updated, are fetched a column ahead of the arithmetic, the shifts once (C and shifts read where they are
// used, whole calls, us: 14 moduli 8000 x 7999 x 200 with beta = 1 926 -> 840, dsyrk 9000 x 200 624 -> 549, 16 moduli dsyrk 5000 x 1024
// 382 -> 352, 8192 x 8192 x 200 794 -> 774; with the shorter tails of oz2_crt_reduce and oz2_digits_to_limbs 765 there, 4096 x 4096 x 1024
// 431 -> 414 in all).
// ---------------------------------------------------------------------------------------------------
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
constexpr int kCrtCols = 16;

// digit held by row rb (0..15) of a 16-row block: rows 0-3 and 8-11 land in lanes 0-31 (digits 0-7), rows 4-7 and
// 12-15 in lanes 32-63 (digits 8-15)
__device__ __forceinline__ constexpr int digit_of_row(int rb) { return ((rb >> 2) & 1) * 8 + (rb >> 3) * 4 + (rb & 3); }

// WIDE: rows 0-3, 8-11, 16 and 17 of a product (registers 0 to 9 of lanes 0-31) and those four rows on (of lanes 32-63)
__device__ __forceinline__ constexpr int wide_digit_of_row(int row) {
  const int e = (row >> 3) * 4 + (row & 3);
  return e < 10 ? ((row >> 2) & 1) * 10 + e : -1;
}

template <int L, bool WIDE>
__global__ void __launch_bounds__(kThreads) crt_mfma_kernel(const uint8_t* __restrict__ planes, int64_t m_pad, int64_t n_pad,
                                                            const int* __restrict__ sa, const int* __restrict__ sb,
                                                            double* __restrict__ C, int64_t ldc, int64_t m, int64_t n,
                                                            const double alpha, const double beta,
                                                            const unsigned long long* __restrict__ skip_flag,
                                                            const int triangle, const Oz2CrtConsts cc, const Oz2CrtDigits dg) {
  if (skip_flag != nullptr && *skip_flag != 0ull) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, half = lane >> 5;
  const int64_t i0 = ((int64_t)blockIdx.y * (kThreads / 64) + wv) * 256 + 4 * lane;  // this thread's four rows
  if (i0 - 4 * lane >= m) return;  // the whole wave (planes are padded to multiples of 256 rows: what it reads exists)
  const int64_t j0 = (int64_t)blockIdx.x * kCrtCols;
  // symmetric product: nothing to do for a wave whose 256 rows x 16 columns lie in the other triangle (dsyrk of order
  // 5000 with inner dimension 1024, whole call: 499 -> 430 us)
  if ((triangle == 1 && i0 - 4 * lane + 255 < j0) || (triangle == 2 && i0 - 4 * lane > j0 + kCrtCols - 1)) return;
  const int N = cc.N;

  constexpr int kWords = WIDE ? 5 : 4, kResidues = 4 * kWords;  // words of four residues
  // first operand: row lane % 32, inner positions 16 (lane / 32) .. + 15; nonzero where the row's block is the half
  const v16i_t zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  v4i_t wop = {0, 0, 0, 0};
  int wop_upper = 0;  // WIDE: word 2 of the second product's, where the first one's has zero
  {
    const int row = lane & 31;
    const int mine = WIDE ? wide_digit_of_row(row) : (row >> 4) == half ? digit_of_row(row & 15) : -1;
#pragma unroll
    for (int d = 0; d < kResidues; ++d) {
      const int* w = reinterpret_cast<const int*>(dg.dig[d]);
      if (mine == d) {
        if constexpr (WIDE) {
          wop = half ? v4i_t{w[3], w[4], 0, 0} : v4i_t{w[0], w[1], w[2], 0};
          wop_upper = half ? w[2] : 0;
        } else {
          wop = v4i_t{w[0], w[1], w[2], w[3]};
        }
      }
    }
  }

  const size_t plane_words = (size_t)n_pad * m_pad / 4;
  const unsigned* src = reinterpret_cast<const unsigned*>(planes) + ((size_t)j0 * m_pad + i0) / 4;
  unsigned nx[kResidues];
  auto fetch = [&](int jj) {
#pragma unroll
    for (int t = 0; t < kResidues; ++t)
      nx[t] = (t < N && j0 + jj < n) ? __builtin_nontemporal_load(src + (size_t)t * plane_words + (size_t)jj * (m_pad / 4)) : 0x80808080u;
  };
  // the shifts of these rows and columns, and C where it is updated, one column ahead like the residues
  int row_shift[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) row_shift[r] = sa[i0 + r];  // sa is padded to m_pad
  const int col_shifts = sb[j0 + (lane & (kCrtCols - 1)) < n ? j0 + (lane & (kCrtCols - 1)) : n - 1];
  auto mine = [&](int r, int64_t j) { return i0 + r < m && !(triangle == 1 && i0 + r < j) && !(triangle == 2 && i0 + r > j); };
  auto all_mine = [&](int64_t j) { return i0 + 4 <= m && (triangle == 0 || (triangle == 1 && i0 >= j) || (triangle == 2 && i0 + 3 <= j)); };
  double old[4] = {0.0, 0.0, 0.0, 0.0};
  auto fetch_c = [&](int jj) {
    const int64_t j = j0 + jj;
    if (beta == 0.0 || j >= n) return;  // C is not read when beta is zero (BLAS convention)
    const double* p = C + i0 + j * ldc;
    if (all_mine(j) && (reinterpret_cast<uintptr_t>(p) & 15) == 0) {
      const double2 lo = *reinterpret_cast<const double2*>(p), hi = *reinterpret_cast<const double2*>(p + 2);
      old[0] = lo.x, old[1] = lo.y, old[2] = hi.x, old[3] = hi.y;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (mine(r, j)) old[r] = p[r];
    }
  };
  fetch(0);
  if (!WIDE) fetch_c(0);
  for (int jj = 0; jj < kCrtCols; ++jj) {
    const int64_t j = j0 + jj;
    if (j >= n) break;  // uniform
    unsigned x[kResidues];
#pragma unroll
    for (int t = 0; t < kResidues; ++t) x[t] = nx[t] ^ 0x80808080u;  // c'' - 128 as signed bytes
    double now[4];
    if (WIDE) fetch_c(jj);  // (and the next residues between the rows: both a column ahead take 145 registers, this 133)
#pragma unroll
    for (int r = 0; r < 4; ++r) now[r] = old[r];
    if (!WIDE && jj + 1 < kCrtCols) {
      fetch(jj + 1);
      fetch_c(jj + 1);
    }
    // words [modulus](4 rows) -> words [row][group of four moduli]
    int y[4][kWords];
#pragma unroll
    for (int g = 0; g < kWords; ++g) {
      const unsigned a = __builtin_amdgcn_perm(x[4 * g + 1], x[4 * g], 0x05010400u);  // x0.b0 x1.b0 x0.b1 x1.b1
      const unsigned b = __builtin_amdgcn_perm(x[4 * g + 1], x[4 * g], 0x07030602u);  // x0.b2 x1.b2 x0.b3 x1.b3
      const unsigned c = __builtin_amdgcn_perm(x[4 * g + 3], x[4 * g + 2], 0x05010400u);
      const unsigned d = __builtin_amdgcn_perm(x[4 * g + 3], x[4 * g + 2], 0x07030602u);
      y[0][g] = (int)__builtin_amdgcn_perm(c, a, 0x05040100u);  // a.lo16 c.lo16
      y[1][g] = (int)__builtin_amdgcn_perm(c, a, 0x07060302u);  // a.hi16 c.hi16
      y[2][g] = (int)__builtin_amdgcn_perm(d, b, 0x05040100u);
      y[3][g] = (int)__builtin_amdgcn_perm(d, b, 0x07060302u);
    }
    const int sbj = __builtin_amdgcn_readlane(col_shifts, jj);
    double out[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int D[kResidues];
      if constexpr (WIDE) {
        const auto s03 = __builtin_amdgcn_permlane32_swap((unsigned)y[r][0], (unsigned)y[r][3], false, false);
        const auto s14 = __builtin_amdgcn_permlane32_swap((unsigned)y[r][1], (unsigned)y[r][4], false, false);
        // (word 3 of the weights is zero)
        const v16i_t lower = __builtin_amdgcn_mfma_i32_32x32x32_i8(wop, v4i_t{(int)s03[0], (int)s14[0], y[r][2], y[r][2]}, zero16, 0, 0, 0);
        const v16i_t upper = __builtin_amdgcn_mfma_i32_32x32x32_i8(half ? v4i_t{wop[0], wop[1], wop_upper, 0} : v4i_t{wop[0], wop[1], 0, 0},
                                                                   v4i_t{(int)s03[1], (int)s14[1], y[r][2], y[r][2]}, zero16, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 10; ++e) {
          // lanes 0-31 keep register e of the first product (digit e) and get the other half's (digit 10 + e); lanes 32-63 have
          // theirs from the second one
          const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)lower[e], (unsigned)upper[e], false, false);
          D[e] = (int)sw[0];
          D[10 + e] = (int)sw[1];
        }
      } else {
        const v16i_t acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wop, v4i_t{y[r][0], y[r][1], y[r][2], y[r][3]}, zero16, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // lanes 0-31 keep register e (digit e) and get the other half's register e (digit 8 + e) in the place of
          // register 8 + e; lanes 32-63 the other way round
          const auto sw = __builtin_amdgcn_permlane32_swap((unsigned)acc[e], (unsigned)acc[8 + e], false, false);
          D[e] = (int)sw[0];
          D[8 + e] = (int)sw[1];
        }
      }
      double S[L];
      oz2_digits_to_limbs<L, kResidues>(D, dg.sinit, S);
      int e2;
      const double xv = oz2_crt_reduce<L>(S, cc, &e2);
      out[r] = ldexp(xv, e2 - row_shift[r] - sbj);
      if (WIDE && r == 1 && jj + 1 < kCrtCols) fetch(jj + 1);
    }
    double* dst = C + i0 + j * ldc;
    if (alpha != 1.0 || beta != 0.0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) out[r] = fma(alpha, out[r], beta == 0.0 ? 0.0 : beta * now[r]);
    }
    if (all_mine(j) && ((reinterpret_cast<uintptr_t>(dst) & 15) == 0)) {
      store_past(dst, out[0], out[1]);
      store_past(dst + 2, out[2], out[3]);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (mine(r, j)) dst[r] = out[r];
    }
  }
}

// C := beta * C (zero without reading C when beta is zero): the k == 0 and alpha == 0 cases
__global__ void __launch_bounds__(kThreads) scale_c_kernel(double* __restrict__ C, int64_t ldc, int64_t m, double beta,
                                                           int triangle) {
  int64_t i = (int64_t)blockIdx.y * kThreads + threadIdx.x;
  const int64_t j = blockIdx.x;
  if (i < m && !(triangle == 1 && i < j) && !(triangle == 2 && i > j)) {
    double* p = C + i + (int64_t)blockIdx.x * ldc;
    *p = beta == 0.0 ? 0.0 : beta * *p;
  }
}

// Does the last-level cache hold the UINT8 planes of a result that the products have just written?  (Whole calls, us, read past it /
// through it: 14 moduli 3001 x 2777 x 200 120 / 107, 1024^3 38.3 / 36.9, 12 moduli dsyrk of order 5000 with 200 152 / 142; 268 MB 16 moduli
// 4000 x 4000 x 600 284 / 293, 210 MB dsyrk of order 5000 with 1024 315 / 323.)
bool planes_cached(const Oz2Plan& plan, const Oz2Layout& lay, int triangle) {
  return plan.N * lay.m_pad * lay.n_pad / (triangle ? 2 : 1) <= OZ2_CACHED_RESULT;
}

template <int L>
double host_crt(const Oz2CrtConsts& cc, const int32_t* cprod) {
  double S[L];
  for (int l = 0; l < L; ++l) S[l] = 0.0;
  for (int t = 0; t < cc.N; ++t) {
    double r = oz2_floor_mod(cprod[t], cc.p[t], cc.inv_p[t], cc.half_inv_p[t]);
    for (int l = 0; l < L; ++l) S[l] = fma(r, cc.w[t][l], S[l]);
  }
  int e2;
  double x = oz2_crt_reduce<L>(S, cc, &e2);
  return ldexp(x, e2);
}

}  // namespace

// From 2^25 elements on, 3/2 of them of a symmetric product: below, a thread's 64 elements leave too few threads for the chip and the
// other kernel wins.  Whole calls with inner dimension 300, us, other / matrix cores: 18 moduli 4096^2 245 / 261, 10 moduli 155 / 159, 18
// moduli 5200 x 5100 455 / 470, 16 moduli 409 / 409, 5800 x 5900 524 / 514, 8192^2 860 / 846 with 200; dsyrk of order 5000 with 1024 and 10
// moduli 214 / 225, 6000 with 16 288 / 295, 7000 384 / 377, 8000 487 / 471.
bool oz2_crt_on_matrix_cores(const Oz2Plan& plan, int64_t m, int64_t n, int residue_u8, int triangle) {
  return residue_u8 && plan.digits.valid && (triangle ? m * n / 3 * 2 : m * n) >= ((int64_t)1 << 25);
}

hipError_t oz2_launch_stage3(int64_t m, int64_t n, double alpha, double beta, double* C, int64_t ldc,
                             const Oz2Plan& plan, const Oz2Layout& lay, char* ws, int residue_u8, int check_flag,
                             int triangle, hipStream_t st) {
  const void* cplanes = ws + lay.off_c;
  const unsigned long long* skip = check_flag ? reinterpret_cast<const unsigned long long*>(ws + lay.off_flags) : nullptr;
  const int* sa = reinterpret_cast<const int*>(ws + lay.off_sa);
  const int* sb = triangle ? sa : reinterpret_cast<const int*>(ws + lay.off_sb);  // symmetric: columns are A's rows
  if (oz2_crt_on_matrix_cores(plan, m, n, residue_u8, triangle)) {
    // at most OZ2_MFMA_N moduli: the accumulation of line 9 on the matrix cores
    const uint8_t* p8 = static_cast<const uint8_t*>(cplanes);
    dim3 g2((unsigned)((n + kCrtCols - 1) / kCrtCols), (unsigned)((m + 1023) / 1024));
    switch (plan.N > 16 ? OZ2_MAX_L : plan.crt.L) {
      case OZ2_MAX_L:  // 17 to 20 moduli: four limbs
        hipLaunchKernelGGL((crt_mfma_kernel<4, true>), g2, dim3(kThreads), 0, st, p8, lay.m_pad, lay.n_pad, sa, sb, C, ldc, m, n, alpha,
                           beta, skip, triangle, plan.crt, plan.digits);
        break;
#define OZ2_CASE(LL)                                                                                                  \
  case LL:                                                                                                            \
    hipLaunchKernelGGL((crt_mfma_kernel<LL, false>), g2, dim3(kThreads), 0, st, p8, lay.m_pad, lay.n_pad, sa, sb, C, ldc, m, \
                       n, alpha, beta, skip, triangle, plan.crt, plan.digits);                                         \
    break;
      OZ2_CASE(1)
      OZ2_CASE(2)
      OZ2_CASE(3)
      OZ2_CASE(4)
#undef OZ2_CASE
      default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  // four rows per thread (eight of UINT8 planes, 64 bytes of C at once, leave few waves for a small result and no more bytes in flight:
  // whole calls, us, eight / four: dtrmm 4096 x 2048 446 / 433, of order 1000 50.6 / 47.7; dsyrk of order 3000 with inner dimension 300
  // 92.7 / 82.9, 4000 with 500 and 18 moduli 201 / 187; 22 moduli 5000 x 5000 x 200 510 / 499, 8192 x 8192 x 200 1220 / 1211)
  constexpr int rows = 4;
  const int64_t per_col = (m + rows - 1) / rows;
  const FastDiv by_col = fast_div((unsigned)per_col);
  const bool cached = planes_cached(plan, lay, triangle);
  // the pieces of a launch are counted below 2^31: results of 2^33 elements and more take several
  const int64_t cols = (((int64_t)1 << 31) - kThreads) / per_col;
  for (int64_t j0 = 0; j0 < n; j0 += cols) {
    const int64_t j1 = n - j0 < cols ? n : j0 + cols;
    const dim3 grid((unsigned)((per_col * (j1 - j0) + kThreads - 1) / kThreads));
    switch (plan.crt.L) {
#define OZ2_CASE(LL)                                                                                                    \
    case LL:                                                                                                              \
      if (residue_u8 && cached)                                                                                           \
        hipLaunchKernelGGL((crt_kernel<LL, true, 4, false>), grid, dim3(kThreads), 0, st, cplanes, lay.m_pad, lay.n_pad, sa, sb, \
                           C, ldc, m, j0, j1, alpha, beta, skip, triangle, (int)per_col, by_col, plan.crt);               \
      else if (residue_u8)                                                                                                \
        hipLaunchKernelGGL((crt_kernel<LL, true, 4, true>), grid, dim3(kThreads), 0, st, cplanes, lay.m_pad, lay.n_pad, sa, sb, \
                           C, ldc, m, j0, j1, alpha, beta, skip, triangle, (int)per_col, by_col, plan.crt);               \
      else                                                                                                                \
        hipLaunchKernelGGL((crt_kernel<LL, false, 4, true>), grid, dim3(kThreads), 0, st, cplanes, lay.m_pad, lay.n_pad, sa,    \
                           sb, C, ldc, m, j0, j1, alpha, beta, skip, triangle, (int)per_col, by_col, plan.crt);           \
      break;
      OZ2_CASE(1)
      OZ2_CASE(2)
      OZ2_CASE(3)
      OZ2_CASE(4)
      OZ2_CASE(5)
#undef OZ2_CASE
      default:
        return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

// Stage 3 on UINT8 residue planes and the FP64 fallback in one launch (general product, full C).
hipError_t oz2_launch_stage3_or_fallback(int transa, int transb, int64_t m, int64_t n, int64_t k, double alpha,
                                         const double* A, int64_t lda, const double* B, int64_t ldb, double beta, double* C,
                                         int64_t ldc, const Oz2Plan& plan, const Oz2Layout& lay, char* ws, hipStream_t st) {
  const void* cplanes = ws + lay.off_c;
  const unsigned long long* flag = reinterpret_cast<const unsigned long long*>(ws + lay.off_flags);
  const int* sa = reinterpret_cast<const int*>(ws + lay.off_sa);
  const int* sb = reinterpret_cast<const int*>(ws + lay.off_sb);
  // two rows per thread up to 2^18 elements, four above: enough threads for the chip, and a short chain in each
  const int rows = m * n <= ((int64_t)1 << 18) ? 2 : 4;
  const int64_t per_col = (m + rows - 1) / rows, threads = per_col * n;
  constexpr int FT = kFallbackSmallTile;
  const int64_t tiles_m = (m + FT - 1) / FT, tiles_n = (n + FT - 1) / FT;
  const int64_t crt_blocks = (threads + kThreads - 1) / kThreads;
  if (threads >= ((int64_t)1 << 31) || crt_blocks + tiles_m * tiles_n >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const FastDiv by_col = fast_div((unsigned)per_col);
  const Oz2FallbackArgs f = {transa, transb, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, tiles_m, 0, 0, 0};
  const dim3 grid((unsigned)(crt_blocks + tiles_m * tiles_n));
  const bool by_four = (plan.N - 1) % 8 < 4, cached = planes_cached(plan, lay, 0);
  switch (plan.crt.L) {
#define OZ2_LAUNCH(LL, R, BATCH, PASS_BY)                                                                                  \
  hipLaunchKernelGGL((crt_or_fallback_kernel<LL, R, BATCH, PASS_BY>), grid, dim3(kThreads), 0, st, cplanes, lay.m_pad, lay.n_pad, sa, \
                     sb, flag, (unsigned)crt_blocks, (int)per_col, by_col, f, plan.crt)
#define OZ2_CASE(LL)                     \
  case LL:                               \
    if (rows == 2 && by_four)            \
      OZ2_LAUNCH(LL, 2, 4, false);       \
    else if (rows == 2)                  \
      OZ2_LAUNCH(LL, 2, 8, false);       \
    else if (by_four && cached)          \
      OZ2_LAUNCH(LL, 4, 4, false);       \
    else if (by_four)                    \
      OZ2_LAUNCH(LL, 4, 4, true);        \
    else if (cached)                     \
      OZ2_LAUNCH(LL, 4, 8, false);       \
    else                                 \
      OZ2_LAUNCH(LL, 4, 8, true);        \
    break;
    OZ2_CASE(1)
    OZ2_CASE(2)
    OZ2_CASE(3)
    OZ2_CASE(4)
    OZ2_CASE(5)
#undef OZ2_CASE
#undef OZ2_LAUNCH
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t oz2_launch_scale_c(int64_t m, int64_t n, double beta, double* C, int64_t ldc, int triangle, hipStream_t st) {
  dim3 grid((unsigned)n, (unsigned)((m + kThreads - 1) / kThreads));
  hipLaunchKernelGGL(scale_c_kernel, grid, dim3(kThreads), 0, st, C, ldc, m, beta, triangle);
  return hipGetLastError();
}

template <int L, int DIGITS>
double host_crt_digits(const Oz2CrtConsts& cc, const Oz2CrtDigits& dg, const uint8_t* res) {
  int D[DIGITS];
  for (int i = 0; i < DIGITS; ++i) {
    int acc = 0;  // what the matrix core computes: signed bytes c'' - 128 against the digits
    for (int t = 0; t < cc.N; ++t) acc += ((int)res[t] - 128) * (int)dg.dig[i][t];
    D[i] = acc;
  }
  double S[L];
  oz2_digits_to_limbs<L, DIGITS>(D, dg.sinit, S);
  int e2;
  double x = oz2_crt_reduce<L>(S, cc, &e2);
  return ldexp(x, e2);
}

double oz2_host_crt_digits_impl(const Oz2CrtConsts& cc, const Oz2CrtDigits& dg, const uint8_t* res) {
  if (cc.N > 16) return host_crt_digits<4, OZ2_MFMA_N>(cc, dg, res);
  switch (cc.L) {
    case 1: return host_crt_digits<1, 16>(cc, dg, res);
    case 2: return host_crt_digits<2, 16>(cc, dg, res);
    case 3: return host_crt_digits<3, 16>(cc, dg, res);
    default: return host_crt_digits<4, 16>(cc, dg, res);
  }
}

double oz2_host_crt_impl(const Oz2CrtConsts& cc, const int32_t* cprod) {
  switch (cc.L) {
    case 1: return host_crt<1>(cc, cprod);
    case 2: return host_crt<2>(cc, cprod);
    case 3: return host_crt<3>(cc, cprod);
    case 4: return host_crt<4>(cc, cprod);
    default: return host_crt<5>(cc, cprod);
  }
}
