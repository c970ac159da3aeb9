// Device and host helpers shared by the INT8 GEMM kernels (oz2_stage2.hip, oz2_stage2_tiles.hip).
#ifndef OZ2_GEMM_H
#define OZ2_GEMM_H

#include "oz2_fast_div.h"
#include "oz2_internal.h"

// 16-byte-per-lane direct load global -> LDS.  The wave writes 1024 contiguous bytes starting at the
// LDS byte address in M0; lane l's 16 bytes come from base + its own 32-bit byte offset.  Written as
// inline assembly so that completion is tracked by the kernels' explicit vmcnt waits (one per k-tile)
// instead of a conservative wait after every load.
__device__ __forceinline__ void load_to_lds_16(const int8_t* base, unsigned voff, unsigned lds_addr) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1"
      :
      : "v"(voff), "s"(base), "s"(lds_addr)
      : "memory", "m0");
}

// The same in two steps, for several loads to one place: M0 once, then loads whose OFFSET counts for the source and for the target.
// Nothing else in the kernel may use M0 between them (build.py looks).
__device__ __forceinline__ void set_lds_target(unsigned lds_addr) { asm volatile("s_mov_b32 m0, %0" : : "s"(lds_addr) : "m0"); }
template <int OFFSET>
__device__ __forceinline__ void load_to_lds_target(const int8_t* base, unsigned voff) {
  static_assert(0 <= OFFSET && OFFSET < 4096, "twelve bits");
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(voff), "s"(base), "n"(OFFSET) : "memory");
}

// s_waitcnt vmcnt(N) only (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// wait_vmcnt<STRICT>, or wait_vmcnt<LOOSE> while i is below `below` (both uniform): one scalar branch, where the compiler
// makes three of the two-sided form.
template <int STRICT, int LOOSE>
__device__ __forceinline__ void wait_vmcnt_unless_below(int i, int below) {
  static_assert(0 <= STRICT && STRICT <= LOOSE && LOOSE < 64, "six bits");
  asm volatile(
      "s_cmp_lt_i32 %0, %1\n\t"
      "s_cbranch_scc1 .Loose%=\n\t"
      "s_waitcnt vmcnt(%2)\n"
      ".Loose%=:\n\t"
      "s_waitcnt vmcnt(%3)"
      :
      : "s"(i), "s"(below), "n"(STRICT), "n"(LOOSE)
      : "memory", "scc");
}

// The triangle of `rows` rows of tiles (triangle 1: lower, 2: upper) laid out as a rectangle of half as many rows (rounded up)
// and one column more (for an even number of them): row y holds the triangle's row rows - 1 - y and, behind it, the
// short row that fills it up.  In: a tile of the rectangle; out: the tile of the triangle.
__device__ __forceinline__ void unfold_triangle(int rows, int triangle, int& tm, int& tn) {
  const int y = tm, x = tn, len = rows - y;
  tm = x < len ? rows - 1 - y : ((rows & 1) ? y - 1 : y);
  tn = x < len ? x : x - len;
  if (triangle == 2) {
    const int swap = tm;
    tm = tn;
    tn = swap;
  }
}
inline void fold_triangle(int rows, int* tiles_m, int* tiles_n) {
  *tiles_n = rows % 2 ? rows : rows + 1;
  *tiles_m = (rows + 1) / 2;
}

// ---------------------------------------------------------------------------------------------------
// Algorithm 1 line 7 in the epilogue of the products: the residue in [0, p) of an INT32 c', as a byte.
//   acc = c' + OZ2_ACC_START modulo 2^32 (the accumulators start there).  As an unsigned word with bytes b3..b0,
//   x = sum_i b_i (2^(8 i) mod p) + ((-OZ2_ACC_START) mod p) is congruent to c' and at most 2^18; one byte dot product
//   forms it on top of the bits of the float 2^23 + e, so that its result read as a float is 2^23 + e + x exactly.
//   With e chosen so that (2^23 + e) / p lies (p + 1) / (2 p) above an integer, the one rounding of
//   fma(2^23 + e + x, 1/p, K) gives 2^23 + floor(x / p) + j (j a constant): the exact quotient plus one half stays
//   1/(2p) away from every tie, further than 1/p's rounding moves it.  j is what makes e + x - (quotient bits) p congruent to
//   x - floor(x / p) p modulo 256, i.e. the low byte of one 16-bit multiply-add is the residue.  j is at least 1 (256 in the
//   place of 0, which only 255 and 241 ask for): the exact sum may lie half a unit below 2^23 + floor(x / p) + j, and below
//   2^23 floats are spaced by halves, so that j = 0 would leave 2^23 - 1/2 there and a residue of x < p one too small.
//   256 needs no quotient (the low byte of x is the residue, and 256 times anything leaves it alone).
//   OZ2_ACC_START is an inline constant of the MFMA (the bits of 1 / (2 pi)) whose lower 22 bits lie near their middle:
//   sums of |c'| < 2^20.8, which is nearly all of them, agree in their upper ten bits whatever their sign, and the
//   matrix cores switch that much less (they run at the card's power limit; against a start at 2^31, GEMM of 26
//   moduli at 8192^3: 10.61 -> 10.47 ms).  It must exceed every |c'|: terms of at most 2^14, so blocks of the inner
//   dimension of at most OZ2_ACC_BLOCK, plus what a reduction between blocks leaves (below 3 p).
// ---------------------------------------------------------------------------------------------------
#define OZ2_ACC_START 0x3e22f983u
#define OZ2_ACC_BLOCK 61440
static_assert((uint64_t)OZ2_ACC_BLOCK * (1 << 14) + 3 * 256 < OZ2_ACC_START, "sums stay positive");

inline Oz2FoldConsts oz2_fold_consts(int p) {
  Oz2FoldConsts c;
  const unsigned u = (unsigned)p, k1 = 256u % u, k2 = k1 * k1 % u, k3 = k2 * k1 % u;
  c.p = p;
  c.inv_p = 1.0f / (float)p;
  c.kpack = (1u % u) | (k1 << 8) | (k2 << 16) | (k3 << 24);
  c.neg_p = (1u << 16) - u;
  const unsigned start = (u - OZ2_ACC_START % u) % u;
  unsigned e = 0, j = 0, above = 0;
  if (u & 1u) {
    const unsigned half = (u + 1u) / 2u;
    e = (half + u - (1u << 23) % u) % u;
    above = ((1u << 23) + e - half) / u;
    unsigned inv = u;  // 1/p modulo 256: each step doubles the number of right bits (p p = 1 modulo 8)
    for (int i = 0; i < 3; ++i) inv *= 2u - u * inv;
    j = (e * inv) & 255u;
    if (j == 0) j = 256;
  }
  c.base = 0x4b000000u + e + start;
  c.offset = (float)((1u << 23) - above - 1u + j);
  c.recip = (unsigned)((((uint64_t)1 << 32) + u / 2u) / u);
  c.half = (1u << 31) / u - OZ2_ACC_START * c.recip;
  return c;
}

// Sums of at most OZ2_SHORT_SUM terms: |c'| <= 2^24.  With M = 2^32 / p + e, |e| <= 1/2, the low word of c' M + 2^31 / p is 2^32 times the
// fraction of c' / p + 1 / (2 p) + c' e / 2^32, and p times that fraction is the residue plus one half, moved by less than
// 2^24 p / 2^33 <= 1/2 (p = 256 has e = 0, 255 below it 255/512) and p / 2^32 for the rounding of the half: the upper word of a product
// with p is the residue.  Two instructions in the place of three, nine cycles of them for the 16-bit multiply-add on a lone wave, and none
// of them a dot product, which waits for the matrix core.
#define OZ2_SHORT_SUM 1024
inline uint8_t oz2_host_short_residue(int32_t product, const Oz2FoldConsts& c) {
  const unsigned low = ((unsigned)product + OZ2_ACC_START) * c.recip + c.half;
  return (uint8_t)(((uint64_t)low * (unsigned)c.p) >> 32);
}
// Four low words -> four residues, one per byte.
__device__ __forceinline__ unsigned oz2_short_residues4(const unsigned* low, unsigned p) {
  const unsigned a = __builtin_amdgcn_perm(__umulhi(low[1], p), __umulhi(low[0], p), 0x0c0c0400u);
  const unsigned b = __builtin_amdgcn_perm(__umulhi(low[3], p), __umulhi(low[2], p), 0x04000c0cu);
  return a | b;
}

// The same for one value on the host, step by step (the 16-bit multiply-add of the device keeps the same low byte).
inline uint8_t oz2_host_fold_residue(int32_t product, const Oz2FoldConsts& c) {
  const unsigned acc = (unsigned)product + OZ2_ACC_START;
  unsigned x = c.base;
  for (int i = 0; i < 4; ++i) x += ((acc >> (8 * i)) & 255u) * ((c.kpack >> (8 * i)) & 255u);
  const unsigned t = __builtin_bit_cast(unsigned, fmaf(__builtin_bit_cast(float, x), c.inv_p, c.offset));
  return (uint8_t)(t * c.neg_p + x);
}

// Four byte sums x (the results of the dot product) -> four residues, one per byte: two of the 16-bit multiply-adds write
// the upper half of a register whose lower half the other two have written, and one byte permutation collects all four.
__device__ __forceinline__ unsigned oz2_fold_residues4(const unsigned* x, const Oz2FoldConsts& c) {
  unsigned t[4], lo, hi;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = __float_as_uint(fmaf(__uint_as_float(x[i]), c.inv_p, c.offset));
  // (one statement: the compiler puts an s_nop between dependent ones; the last result can be read two instructions later, which it sees to)
  asm("v_mad_u16 %0, %2, %6, %7\n\tv_mad_u16 %1, %4, %6, %9\n\t"
      "v_mad_u16 %0, %3, %6, %8 op_sel:[0,0,0,1]\n\tv_mad_u16 %1, %5, %6, %10 op_sel:[0,0,0,1]"
      : "=&v"(lo), "=&v"(hi)
      : "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(c.neg_p), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]));
  return __builtin_amdgcn_perm(hi, lo, 0x06040200u);
}

// The constants in vector registers: an operand from a scalar register costs an instruction a cycle.
__device__ __forceinline__ unsigned to_vector(unsigned v) {
  unsigned r;
  asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
  return r;
}
__device__ __forceinline__ Oz2FoldConsts in_vector_registers(const Oz2FoldConsts& c) {
  Oz2FoldConsts v = c;
  v.kpack = to_vector(c.kpack);
  v.base = to_vector(c.base);
  v.neg_p = to_vector(c.neg_p);
  v.recip = to_vector(c.recip);
  v.half = to_vector(c.half);
  v.p = (int)to_vector((unsigned)c.p);
  v.inv_p = __uint_as_float(to_vector(__float_as_uint(c.inv_p)));
  v.offset = __uint_as_float(to_vector(__float_as_uint(c.offset)));
  return v;
}

#endif
