// Element-wise arithmetic of Ozaki scheme II in FP64 operations whose results are exact by construction.
// Every function is __host__ __device__: the kernels use them, and the same source compiled for the host
// backs the unit tests of the exactness arguments written next to each step.
#ifndef OZ2_MATH_H
#define OZ2_MATH_H

#include <hip/hip_runtime.h>
#include <math.h>

#include "oz2_internal.h"

#define OZ2_HD __host__ __device__ __forceinline__

// ---------------------------------------------------------------------------------------------------
// Algorithm 1 lines 2-5 for one element.
//   x = trunc(a * 2^shift) is an integer-valued double (|x| < 2^kappa, possibly far above 2^53: its low
//   bits are zero then).  Split x = x2*2^64 + x1*2^32 + x0 with integer parts of the same sign
//   (|x1|,|x0| < 2^32); then  y_t = x2*c64_t + x1*c32_t + x0  is congruent to x modulo p_t, exact in
//   FP64 and below 2^51 in magnitude, so one rounded quotient gives the symmetric residue exactly:
//   |y/p * 2^-52| < 1/(2p) is the distance of y/p from the nearest rounding tie for odd p.  For
//   p = 256 a tie can occur and yields +128, which wraps to -128 in INT8 (Section 3.1).
// ---------------------------------------------------------------------------------------------------
struct Oz2Split {
  double x2, x1, x0;
};

template <bool TWO_LEVEL>
OZ2_HD Oz2Split oz2_scale_trunc_split(double a, int shift) {
  Oz2Split s;
  double x = trunc(ldexp(a, shift));
  if (TWO_LEVEL) {
    s.x2 = trunc(x * 0x1p-64);
    double rem = fma(-s.x2, 0x1p64, x);
    s.x1 = trunc(rem * 0x1p-32);
    s.x0 = fma(-s.x1, 0x1p32, rem);
  } else {
    s.x2 = 0.0;
    s.x1 = trunc(x * 0x1p-32);
    s.x0 = fma(-s.x1, 0x1p32, x);
  }
  return s;
}

// Two elements side by side.  The quotient q = rint(y/p) is read off the low bits of y/p + 1.5 * 2^52, and the residue
// y - q p, of which only the last 16 bits matter (it lies in [-128, 128]), is formed from the last 16 bits of x0, x1,
// x2 and q, both elements in one register.  Per element and modulus two FP64 instructions and 1.5 others (the rounding,
// the FP64 remainder and its conversion to an integer took five and more to pack the byte: 33 cycles against 18).
typedef unsigned short oz2_u16x2 __attribute__((ext_vector_type(2)));
#define OZ2_ROUND 0x1.8p52  // added to |v| < 2^51, its sum with v ends in the bits of the integer nearest to v

OZ2_HD unsigned oz2_low_word(double v) {
#ifdef __HIP_DEVICE_COMPILE__
  return (unsigned)__double2loint(v);
#else
  return (unsigned)__builtin_bit_cast(unsigned long long, v);
#endif
}
OZ2_HD unsigned oz2_low_halves(unsigned hi, unsigned lo) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
#else
  return (lo & 0xffffu) | (hi << 16);
#endif
}
// byte 0 and byte 2 of two words -> one word
OZ2_HD unsigned oz2_even_bytes(unsigned hi, unsigned lo) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_perm(hi, lo, 0x06040200u);
#else
  return (lo & 0xffu) | ((lo >> 8) & 0xff00u) | ((hi & 0xffu) << 16) | ((hi << 8) & 0xff000000u);
#endif
}
OZ2_HD oz2_u16x2 oz2_halves(double a, double b) {  // last 16 bits of two integer-valued doubles below 2^51
  return __builtin_bit_cast(oz2_u16x2, oz2_low_halves(oz2_low_word(b + OZ2_ROUND), oz2_low_word(a + OZ2_ROUND)));
}

template <bool TWO_LEVEL>
struct Oz2SplitPair {
  Oz2Split a, b;
  oz2_u16x2 x0, x1, x2;
};
template <bool TWO_LEVEL>
OZ2_HD Oz2SplitPair<TWO_LEVEL> oz2_split_pair(double a, double b, int shift) {
  Oz2SplitPair<TWO_LEVEL> s;
  s.a = oz2_scale_trunc_split<TWO_LEVEL>(a, shift);
  s.b = oz2_scale_trunc_split<TWO_LEVEL>(b, shift);
  s.x0 = oz2_halves(s.a.x0, s.b.x0);
  s.x1 = oz2_halves(s.a.x1, s.b.x1);
  s.x2 = TWO_LEVEL ? oz2_halves(s.a.x2, s.b.x2) : oz2_u16x2{0, 0};
  return s;
}

template <bool TWO_LEVEL>
OZ2_HD double oz2_rounded_quotient(const Oz2Split& s, const Oz2ConvMod& m) {
  double y = fma(s.x1, m.c32, s.x0);
  if (TWO_LEVEL) y = fma(s.x2, m.c64, y);
  return fma(y, m.inv_p, OZ2_ROUND);
}

// symmetric residues of both elements as 16-bit integers
template <bool TWO_LEVEL>
OZ2_HD oz2_u16x2 oz2_residue_pair(const Oz2SplitPair<TWO_LEVEL>& s, const Oz2ConvMod& m) {
  const oz2_u16x2 q =
      __builtin_bit_cast(oz2_u16x2, oz2_low_halves(oz2_low_word(oz2_rounded_quotient<TWO_LEVEL>(s.b, m)),
                                                   oz2_low_word(oz2_rounded_quotient<TWO_LEVEL>(s.a, m))));
  oz2_u16x2 r = s.x1 * __builtin_bit_cast(oz2_u16x2, m.c32_h) + s.x0;
  if (TWO_LEVEL) r = s.x2 * __builtin_bit_cast(oz2_u16x2, m.c64_h) + r;
  return q * __builtin_bit_cast(oz2_u16x2, m.neg_p_h) + r;
}

// The same of a two-level split for kernels that hold many elements per thread: the last 16 bits of x0 + x1 c32 are read off
// that sum, modulus by modulus, in the place of those of x0 and x1 kept in registers; without KEEP_X2 those of x2 are
// formed anew too.  One or two FP64 instructions more per element and modulus, 16 to 24 registers less: what decides whether four
// waves share a SIMD or three.
template <bool KEEP_X2>
OZ2_HD oz2_u16x2 oz2_residue_pair_lean(const Oz2SplitPair<true>& s, const Oz2ConvMod& m) {
  const double ta = fma(s.a.x1, m.c32, s.a.x0), tb = fma(s.b.x1, m.c32, s.b.x0);  // below 2^40
  const double qa = fma(fma(s.a.x2, m.c64, ta), m.inv_p, OZ2_ROUND), qb = fma(fma(s.b.x2, m.c64, tb), m.inv_p, OZ2_ROUND);
  oz2_u16x2 x2 = s.x2;
  if (!KEEP_X2) {
    double round = OZ2_ROUND;
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(round));  // (otherwise the compiler forms them once and keeps them)
#endif
    x2 = __builtin_bit_cast(oz2_u16x2, oz2_low_halves(oz2_low_word(s.b.x2 + round), oz2_low_word(s.a.x2 + round)));
  }
  const oz2_u16x2 q = __builtin_bit_cast(oz2_u16x2, oz2_low_halves(oz2_low_word(qb), oz2_low_word(qa)));
  const oz2_u16x2 r = x2 * __builtin_bit_cast(oz2_u16x2, m.c64_h) + oz2_halves(ta, tb);
  return q * __builtin_bit_cast(oz2_u16x2, m.neg_p_h) + r;
}
OZ2_HD unsigned oz2_pack_pairs(oz2_u16x2 lo, oz2_u16x2 hi) {  // low bytes of four 16-bit values
  return oz2_even_bytes(__builtin_bit_cast(unsigned, hi), __builtin_bit_cast(unsigned, lo));
}

// ---------------------------------------------------------------------------------------------------
// Section 4.1, INT8-product bound: ceil(|a| 2^sh) with sh = 5 - floor(log2 of the vector's maximum), an
// integer in [0, 64] that bounds |a| 2^sh from above.  The scaling is exact unless it underflows to zero,
// and the ceiling of any positive value is at least one.
// ---------------------------------------------------------------------------------------------------
OZ2_HD int oz2_bound6(double a, int sh) {
  double q = ceil(ldexp(fabs(a), sh));
  if (a != 0.0 && q == 0.0) q = 1.0;
  return (int)q;
}

// ---------------------------------------------------------------------------------------------------
// Algorithm 1 line 7: c'' = c' - floor(c'/p) p for an INT32 c', as a double in [0, p).
//   floor((c' + 1/2)/p) == floor(c'/p) and (c' + 1/2)/p stays 1/(2p) away from every integer, far more
//   than the rounding error 2^31/p * 2^-52 of the fused multiply-add, so the floor is exact.
// ---------------------------------------------------------------------------------------------------
OZ2_HD double oz2_floor_mod(int c, double p, double inv_p, double half_inv_p) {
  double x = (double)c;
  double q = floor(fma(x, inv_p, half_inv_p));
  return fma(-q, p, x);
}

// ---------------------------------------------------------------------------------------------------
// Algorithm 1 lines 8-10 and the rounding of line 11.
//   Input: S[l] = sum_t c''_t * w_{t,l} (integers below 2^53, exact), i.e. Y = sum_l S[l] 2^(40 l).
//   Output: the double nearest to X = Y mod M (symmetric, Section 2.1) as r * 2^e2.
//   Steps: Q = rint(Y/M) from a floating estimate; T[l] = S[l] - Q*m_l exactly; if the estimate is too
//   close to a half-integer to trust Q, X is compared with M/2 exactly on its digits; carries are
//   propagated so that X = sum_l D[l] 2^(40 l) with |D[l]| <= 2^39 below the top digit; the top three
//   nonzero-led digits are rounded once with the remaining digits acting as a sticky term.
// ---------------------------------------------------------------------------------------------------
template <int L>
OZ2_HD void oz2_carry(double* T) {
#pragma unroll
  for (int l = 0; l + 1 < L; ++l) {
    double c = rint(T[l] * 0x1p-40);
    T[l] = fma(-c, 0x1p40, T[l]);
    T[l + 1] += c;
  }
}

// ---------------------------------------------------------------------------------------------------
// Digit route to the same S[l] (matrix-core CRT kernel): D[i] = sum_t c''_t dig[i][t] for the balanced base-256
// digits of the weights in the symmetric range, sixteen, or twenty above 16 moduli, |D[i]| <= 20 * 255 * 128 < 2^20, so that
//   Y' = sum_i D[i] 256^i  is congruent to  Y = sum_t c''_t W_t  modulo M,  |Y'| <= 2^12 M.
// Limb l collects the digits 5 l .. 5 l + 4 (the top limb all that remain): integers below 2^53, exact.  In a
// top limb with few digits in use the upper D[i] are zero (|Ws| <= M/2 < 2^(40 L - 1)).
// ---------------------------------------------------------------------------------------------------
template <int L, int DIGITS>
OZ2_HD void oz2_digits_to_limbs(const int* D, const double* start, double* S) {
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int first = 5 * l, last = l + 1 < L ? 5 * l + 4 : DIGITS - 1;
    // (two digits at a time as an integer below 2^29: a shift and add in the place of a conversion and an FP64 instruction)
    double v = (last - first) % 2 == 0 ? (double)D[last] : (double)(D[last] * 256 + D[last - 1]);
#pragma unroll
    for (int i = last - 1 - (last - first) % 2; i > first; i -= 2) v = fma(v, 65536.0, (double)(D[i] * 256 + D[i - 1]));
    S[l] = v + start[l];  // the digit sums were formed on c'' - 128: start holds 128 sum_t dig in limb form
  }
}

template <int L>
OZ2_HD double oz2_crt_reduce(const double* S, const Oz2CrtConsts& cc, int* e2) {
  double yest = 0.0;
#pragma unroll
  for (int l = L - 1; l >= 0; --l) yest = fma(S[l], cc.rinv[l], yest);
  double Q = rint(yest);
  double frac = yest - Q;

  constexpr int LP = L < 3 ? 3 : L;
  double D[LP];
#pragma unroll
  for (int l = 0; l < LP; ++l) D[l] = l < L ? fma(-Q, cc.mlimb[l], S[l]) : 0.0;

  if (fabs(frac) > 0.4999990463256836) {  // 0.5 - 2^-20: the estimate (error < 2^-36) cannot decide
    double sgn = frac > 0.0 ? 1.0 : -1.0;
    double U[L];
#pragma unroll
    for (int l = 0; l < L; ++l) U[l] = sgn * D[l] - cc.mhalf[l];
    oz2_carry<L>(U);
    double lead = 0.0;  // highest nonzero digit of sgn*X - M/2
#pragma unroll
    for (int l = 0; l < L; ++l)
      if (U[l] != 0.0) lead = U[l];
    if (lead > 0.0 || (lead == 0.0 && sgn > 0.0)) {  // X outside [-M/2, M/2)
      Q += sgn;
#pragma unroll
      for (int l = 0; l < L; ++l) D[l] = fma(-Q, cc.mlimb[l], S[l]);
    }
  }
  oz2_carry<L>(D);

  double dh = D[2], dm = D[1], lo = D[0];
  int shift = 0;
  if (L == 4 && cc.joined) {
    // |X| < 2^146: the top two digits joined, dh 2^80 + dm 2^40 + lo = X with integers dh and dm.  What rounding dh loses is below
    // 2^13 and goes to the digit below, where it is exact.
    const double u = D[LP - 1] * 0x1p40;
    dh = u + D[2];                             // |u| >= 2^40 > |D[2]| or u == 0: Fast2Sum
    dm = fma(D[2] - (dh - u), 0x1p40, D[1]);
  } else if (L > 3) {
    // window of three digits led by the highest nonzero one (or the lowest three)
    double rest = 0.0;
#pragma unroll
    for (int w = 3; w < LP; ++w) {
      if (D[w] != 0.0) {
        dh = D[w];
        dm = D[w - 1];
        lo = D[w - 2];
        double rr = 0.0;
#pragma unroll
        for (int i = 0; i <= w - 3; ++i)
          if (D[i] != 0.0) rr = D[i];
        rest = rr;
        shift = OZ2_LIMB_BITS * (w - 2);
      }
    }
    // the digits below the window only matter through their sign: move its last one by a quarter unit
    lo += rest > 0.0 ? 0.25 : (rest < 0.0 ? -0.25 : 0.0);
  }
  const double hi = dh * 0x1p80, mid = dm * 0x1p40;
  const double a = hi + mid;          // |hi| >= |mid| (2^80 > 2^79, or dh >= 2^53 where dm is above 2^39) or hi == 0: Fast2Sum
  const double b = mid - (a - hi);
  // b != 0: |b| >= 2^40 > 2|lo|, so lo can only break an exact tie of a + b; nudge b by one part in 2^52
  const double nudged = fma(fabs(b), copysign(lo != 0.0 ? 0x1p-52 : 0.0, lo), b);
  const double tail = b != 0.0 ? nudged : lo;
  *e2 = shift;
  return a + tail;
}

#endif
