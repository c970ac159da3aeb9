// Stage 2 of Ozaki scheme II on gfx950: Algorithm 1 line 6, C'_t = A'_t B'_t for every modulus t with
// INT8 operands and INT32 accumulation on the matrix cores (v_mfma_i32_16x16x64_i8).
//
// Operand layout (written by stage 1): each residue plane is stored in blocks of 256 rows x 64 bytes of
// the inner dimension, every block contiguous (16 KiB): element (row, l) of plane t lives at
//   ((t*rows_pad + 256*(row/256)) * k_pad) + (l/64)*16384 + (row%256)*64 + (l%64).
// Rows and the inner dimension are zero padded to the tile sizes, so the kernel has no edge cases, and
// every global -> LDS copy of a k-tile reads contiguous kilobytes (a row-major plane with a power-of-two
// pitch would hit the same L2 channels with all 256 rows of a tile).  Output plane t holds element (i,j)
// at (j*m_pad + i), i contiguous: either the INT32 product itself, or (RESIDUE_U8) its residue in [0, p_t) as
// one byte (Algorithm 1 line 7 taken in the epilogue; four times less to write here and to read in stage 3).
//
// One workgroup (4 waves, one per SIMD) computes a 256 x 256 tile of one modulus.  Each wave owns a
// 128 x 128 sub-tile = 8 x 8 MFMA tiles of 16 x 16 (256 accumulator registers).  The inner dimension is
// walked in k-tiles of 64 bytes through a ring of four LDS stages (32 KiB each).  Both operands of a
// k-tile are copied global -> LDS with 16-byte direct loads (no VGPR staging).  LDS rows are 64 bytes; the
// 16-byte chunk index is XOR-swizzled with two bits of the row so that the 16 rows read together by a
// ds_read_b128 fall on 16 different bank groups (measured: no bank conflicts): bits 2..3 for the columns of B', whose MFMA tiles
// are sixteen neighbouring rows of the plane, bits 4..5 for A', whose tile x of a group of four is the rows 16 q + 4 x + (0..3),
// q = 0..3, of 64.  A lane's words of four such tiles then are sixteen neighbouring rows of C', which it stores at once; with
// neighbouring rows in a tile four exchanges between lanes per sixteen bytes did that (9 cycles each;
// whole calls, us, 18 moduli 8192 x 8192 x 1024 1711 -> 1690, 16 moduli 4096^3 1044 -> 1041, dsyrk 5000 x 1024 344 -> 340).
//
// Which matrix instruction: under the card's power cap the products of 16 x 16 x 64 run at 4.0 POP/s on random operands with no
// memory traffic, those of 32 x 32 x 32 at 3.5 (the larger tile moves twice the accumulator bytes per operation through the
// register file).  Whole calls, ms, 16384^3 with 16 moduli in the Strassen form 53.5 -> 49.9, 8192^3 even at 7.63, 18 moduli
// 8192 x 8192 x 1024 1.78 -> 1.74, 4096^3 1.134 -> 1.094.
//
// Schedule of one k-tile (64 MFMAs: tile rows 0-3 against all eight columns, then rows 4-7): there is one set of fragments, each
// read again for the next k-tile after its last product.  During the first half rows 4-7 and the last column arrive; at
// the start of the second one vmcnt wait + barrier makes the NEXT k-tile visible to all waves; during the rest its rows 0-3 and columns
// 0-6 are read and the 8 direct loads that refill the stage freed by the barrier are issued, spread out so that no queue
// fills up.  A product occupies the matrix core for 16 cycles and any other instruction the issue of the one wave for four or five, so
// not more than two or three stand between two products: 130 instructions per k-tile, one M0 for four direct loads, scalar arithmetic in
// the first half (175, six of them around every direct load, before: 8192^3 7.64 -> 7.00 ms a call, 16384^3 49.9 -> 47.9, 4096^3 1.094 -> 1.050).
//
// INT32 accumulation is exact for fewer than 2^17 terms (Section 3.1).  For longer inner dimensions the
// accumulators are reduced modulo p_t every `kblock` bytes of k (kblock <= 65536, UINT8 residues: 61440), which keeps them below
// 2^31 and leaves the residue of the product unchanged.
//
// The 1-D grid is remapped so that the 32 workgroups resident on an XCD (workgroup id mod 8) form an
// 8 x 4 block of tiles and share A' and B' panels in that XCD's L2.  When the tile grid is a multiple of
// 16 x 16 the eight XCDs additionally work on the eight 8 x 4 sub-blocks of one 16 x 16 super-block at the
// same time, so that panels re-read by several XCDs come from the shared last-level cache instead of HBM
// (measured: same L2 miss count, higher clock under the power cap, +6 % throughput).  Tile grids that are
// multiples of 8 x 4 only (24 x 24, 40 x 40 tiles ...) get the same effect from a list of all 8 x 4 sub-blocks, of
// which the eight XCDs take eight consecutive entries per round (a kernel instantiation of its own, LIST_ORDER,
// so that the tile decoding of the other orders stays as it is; measured: GEMM -2 % at 6144^3, -4 % at 10240^3).
// Otherwise each XCD walks its own contiguous range of tiles in 8-tile-tall column groups.
//
// General products are launched with one workgroup per compute unit; each walks the work indices of its slot in
// launch order (so the mapping above is unchanged).  The ring of LDS stages runs on from tile to tile: every
// iteration of the main loop fetches the k-tile NS - 1 ahead of the one it multiplies, and when that runs past the
// end of the tile it fetches the first k-tiles of the workgroup's next tile, so the copies of a new tile cost no
// time of their own at the tile boundary (measured against issuing them after the main loop, before the
// epilogue: GEMM -9 % at k = 1024, -5 % at 4096^3, -1 % at 8192^3, even at 16384^3 where the power cap decides).
// The loop has one body for every iteration and the same number of copies in flight at every wait.
//
// Structured products: for the symmetric product op(A) op(A)^T both operands are A's planes and only the tiles of one
// triangle are launched (in the super-block order: those of the other one return at once); for a triangular operand a tile
// walks only the k-tiles up to or from its diagonal block.
#include <type_traits>

#include "oz2_gemm.h"
#include "oz2_scan_finish.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int BM = OZ2_TILE_M, BN = OZ2_TILE_N, BK = OZ2_TILE_K;
static_assert(BM == 256 && BN == 256 && BK == 64, "the kernel below is written for 256 x 256 x 64 tiles");
constexpr int kThreads = 256;
constexpr int NS = 4;                            // LDS stages
constexpr int kStageBytes = (BM + BN) * BK;      // 32 KiB: A tile then B tile
constexpr int kLdsBytes = NS * kStageBytes;
static_assert((kLdsBytes & (kLdsBytes - 1)) == 0, "the ring of stages wraps by a mask");
constexpr int kLoads = 8;                        // direct loads per wave per k-tile
constexpr int kGroupM = 8;
// The product behind which the barrier stands: the first ones of the second half cover the arrival of the last fragments.
constexpr int kSyncAt = 33;
// The tile orders below are written for the eight accelerator dies (XCDs) of the MI355X, on which the hardware
// places workgroup i of a launch on die i % 8.
constexpr int kXcds = 8;
constexpr int kStores = 16;                      // stores per wave of an epilogue (UINT8; the INT32 one has more)

struct GemmArgs {
  const int8_t* a;
  const int8_t* b;
  int* c;
  int64_t m_pad, n_pad, k_pad;
  int tiles_m, tiles_n, num_moduli;
  int total, chunk;        // work items, and items per XCD
  int superblock;          // 1: tiles_m and tiles_n are multiples of 16, use the super-block order
  int ktiles;              // k_pad / BK
  int ktiles_per_block;    // k-tiles between modular reductions of the accumulators
  int triangle;            // 0: all tiles; 1: only tiles with tm >= tn (lower); 2: only tm <= tn (upper)
  int folded;              // tile rows of the triangle when tiles_m x tiles_n is its rectangle (unfold_triangle), else 0
  int krange;              // triangular operand: which k-tiles of a tile can be nonzero (see OZ2_KRANGE_*)
  const unsigned long long* skip_flag;  // if not null and nonzero on the device: the products are not needed
  Oz2ScanFinish fin;                    // reports of stage 1 that workgroup 0 turns into the flag word
  int fin_stops;                        // 1: every workgroup looks at the reports and stops when there is one
  unsigned long long* xcd_sync;         // one counter per XCD (zero at launch), or null: no round sync
  int full_rounds;                      // rounds in which every workgroup slot has a tile
  int sync_spins;                       // bound of one wait of the round synchronisation, in polls of the counter
  FastDiv per_modulus;                  // planes per modulus: plane u is reduced modulo number u / per_modulus
  FastDiv div_plane;                    // tiles, sub-blocks or super-blocks of a plane
  FastDiv div_rows, div_cols;           // sub-blocks or super-blocks down a column and along a row of them
  FastDiv div_group, div_last;          // tiles of a group of kGroupM tile rows, tile rows of the last group
  Oz2FoldConsts fold[OZ2_MAX_N];        // residue epilogue and reduction between k-blocks, per modulus
};

// Any representative of c modulo p with |result| <= 3p is enough between k-blocks: the final residue is
// taken in stage 3.  The quotient is estimated in FP32 (error below two units).
__device__ __forceinline__ int reduce_mod(int c, int p, float inv_p) {
  int q = (int)rintf((float)c * inv_p);
  return c - q * p;
}

// ---- The 256 accumulators of a lane live in registers by name: MFMA tile (x, y) of the wave's 8 x 8, T = x + 8 y, in
// the ordinary registers v[112 + 4 T ...] for T < kVgprTiles and in the accumulation registers a[4 T ...] for the
// others.  An ordinary instruction reads the former directly, the latter only through a move of eight cycles, and
// of the 256 ordinary registers the kernel's own code needs fewer than 112 (build.py refuses a build in which the compiler
// uses a register named here, or scratch memory; amdgpu_num_vgpr keeps it to them, and named_accumulators tells it that the kernel
// has them).  (As variables the accumulators were copied through ordinary
// registers and scratch memory wherever the main loop meets the code around it: up to 256 moves per tile and 20 to 1200
// bytes of scratch per lane, depending on the form of the loop.)
// What the compiler does not see is the distance an MFMA needs to a reader of its result (settle_acc).  Operands come
// from LDS reads, whose arrival it waits for, and the next MFMA on the same accumulators is 63 others away.
constexpr int kVgprTiles = 32;
template <int T>
struct Acc {
  static constexpr bool kV = T < kVgprTiles;
  static constexpr int kReg = kV ? 112 + 4 * T : 4 * T;
  /* acc := acc + a b */
  static __device__ __forceinline__ void add(const v4i& a, const v4i& b) {
    if constexpr (kV)
      asm volatile("v_mfma_i32_16x16x64_i8 v[%2:%3], %0, %1, v[%2:%3]" : : "v"(a), "v"(b), "n"(kReg), "n"(kReg + 3));
    else
      asm volatile("v_mfma_i32_16x16x64_i8 a[%2:%3], %0, %1, a[%2:%3]" : : "v"(a), "v"(b), "n"(kReg), "n"(kReg + 3));
  }
  /* acc := start + a b */
  template <bool RESIDUE_U8>
  static __device__ __forceinline__ void start(const v4i& a, const v4i& b) {
    if constexpr (kV && RESIDUE_U8)
      asm volatile("v_mfma_i32_16x16x64_i8 v[%2:%3], %0, %1, 0.15915494" : : "v"(a), "v"(b), "n"(kReg), "n"(kReg + 3));
    else if constexpr (kV)
      asm volatile("v_mfma_i32_16x16x64_i8 v[%2:%3], %0, %1, 0" : : "v"(a), "v"(b), "n"(kReg), "n"(kReg + 3));
    else if constexpr (RESIDUE_U8)
      asm volatile("v_mfma_i32_16x16x64_i8 a[%2:%3], %0, %1, 0.15915494" : : "v"(a), "v"(b), "n"(kReg), "n"(kReg + 3));
    else
      asm volatile("v_mfma_i32_16x16x64_i8 a[%2:%3], %0, %1, 0" : : "v"(a), "v"(b), "n"(kReg), "n"(kReg + 3));
  }
  static __device__ __forceinline__ unsigned read(int e) {
    unsigned v;
    if constexpr (kV)
      asm volatile("v_mov_b32 %0, v[%1+%2]" : "=v"(v) : "n"(kReg), "n"(e));
    else
      asm volatile("v_accvgpr_read_b32 %0, a[%1+%2]" : "=v"(v) : "n"(kReg), "n"(e));
    return v;
  }
  static __device__ __forceinline__ void write(int e, unsigned v) {
    if constexpr (kV)
      asm volatile("v_mov_b32 v[%1+%2], %0" : : "v"(v), "n"(kReg), "n"(e));
    else
      asm volatile("v_accvgpr_write_b32 a[%1+%2], %0" : : "v"(v), "n"(kReg), "n"(e));
  }
  /* oz2_fold_sum; its result can be read three instructions later (settle_sums) */
  static __device__ __forceinline__ unsigned fold_sum(int e, unsigned kpack, unsigned base) {
    unsigned v;
    if constexpr (kV)
      asm volatile("v_dot4_u32_u8 %0, v[%3+%4], %1, %2" : "=&v"(v) : "v"(kpack), "v"(base), "n"(kReg), "n"(e));
    else
      asm volatile("v_accvgpr_read_b32 %0, a[%3+%4]\n\tv_dot4_u32_u8 %0, %0, %1, %2" : "=&v"(v) : "v"(kpack), "v"(base), "n"(kReg), "n"(e));
    return v;
  }
  /* the low words of (acc) (recip) + half, in one statement: the compiler puts an s_nop between several */
  static __device__ __forceinline__ void low_words(unsigned* low, unsigned recip, unsigned long long half) {
    unsigned long long w[4];
    if constexpr (kV) {
      asm volatile(
          "v_mad_u64_u32 %0, vcc, v[%6+0], %4, %5\n\tv_mad_u64_u32 %1, vcc, v[%6+1], %4, %5\n\t"
          "v_mad_u64_u32 %2, vcc, v[%6+2], %4, %5\n\tv_mad_u64_u32 %3, vcc, v[%6+3], %4, %5"
          : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
          : "v"(recip), "v"(half), "n"(kReg)
          : "vcc");
    } else {
      unsigned t[4];
      asm volatile(
          "v_accvgpr_read_b32 %4, a[%10+0]\n\tv_accvgpr_read_b32 %5, a[%10+1]\n\t"
          "v_accvgpr_read_b32 %6, a[%10+2]\n\tv_accvgpr_read_b32 %7, a[%10+3]\n\t"
          "v_mad_u64_u32 %0, vcc, %4, %8, %9\n\tv_mad_u64_u32 %1, vcc, %5, %8, %9\n\t"
          "v_mad_u64_u32 %2, vcc, %6, %8, %9\n\tv_mad_u64_u32 %3, vcc, %7, %8, %9"
          : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3])
          : "v"(recip), "v"(half), "n"(kReg)
          : "vcc");
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) low[e] = (unsigned)w[e];
  }
};
#define OZ2_TEN(R, N) R #N "0", R #N "1", R #N "2", R #N "3", R #N "4", R #N "5", R #N "6", R #N "7", R #N "8", R #N "9"
__device__ __forceinline__ void named_accumulators() {
  asm volatile("" : : : "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", OZ2_TEN("v", 12), OZ2_TEN("v", 13),
               OZ2_TEN("v", 14), OZ2_TEN("v", 15), OZ2_TEN("v", 16), OZ2_TEN("v", 17), OZ2_TEN("v", 18), OZ2_TEN("v", 19),
               OZ2_TEN("v", 20), OZ2_TEN("v", 21), OZ2_TEN("v", 22), "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237",
               "v238", "v239", "a128", "a129", OZ2_TEN("a", 13), OZ2_TEN("a", 14), OZ2_TEN("a", 15), OZ2_TEN("a", 16),
               OZ2_TEN("a", 17), OZ2_TEN("a", 18), OZ2_TEN("a", 19), OZ2_TEN("a", 20), OZ2_TEN("a", 21), OZ2_TEN("a", 22),
               OZ2_TEN("a", 23), OZ2_TEN("a", 24), "a250", "a251", "a252", "a253", "a254", "a255");
}
#undef OZ2_TEN
static_assert(OZ2_ACC_START == 0x3e22f983u, "the bits of 1 / (2 pi), an inline constant of the instruction");

// The wait between the last MFMA and the first use of a result by another instruction (19 states are enough for the longest ones),
// and between a write by another instruction and the next MFMA.
__device__ __forceinline__ void settle_acc() { asm volatile("s_nop 15\n\ts_nop 3"); }
// The wait between a byte dot product and the first use of its result by another kind of instruction.
__device__ __forceinline__ void settle_sums(unsigned (&x)[16]) {
  asm volatile("s_nop 2"
               : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]), "+v"(x[8]),
                 "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]));
  asm volatile("" : "+v"(x[15]));
}

// Calls f(integral_constant<int, 0>) .. f(integral_constant<int, COUNT - 1>).
template <int COUNT, int I = 0, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < COUNT) {
    f(std::integral_constant<int, I>());
    unrolled<COUNT, I + 1>(f);
  }
}

// Operands of a k-tile: sixteen rows x 64 bytes each, lane l holds 16 bytes (inner positions 16 (l / 16) ..) of row l % 16.
struct Frag {
  v4i a[8], b[8];
};

// What one workgroup needs to know about a unit of work.
struct Tile {
  int t, tm, tn;
  int ktiles;            // k-tiles this tile walks, at least 1
  const int8_t* a_wave;  // first byte this wave copies of the tile's first k-tile of A'
  const int8_t* b_wave;  // same for B'
  bool valid;            // false: nothing to compute for this work index
};

// Work index -> tile.  `slot` counts workgroup slots in launch order: slot % 8 is the XCD a workgroup of a plain
// launch would land on, and the persistent loop keeps that residue (its stride is a multiple of 8).
template <bool LIST_ORDER>
__device__ __forceinline__ Tile decode_tile(const GemmArgs& g, int slot, int wv) {
  Tile T;
  T.valid = false;
  T.ktiles = 0;
  T.a_wave = T.b_wave = nullptr;
  T.t = T.tm = T.tn = 0;
  if (slot >= g.chunk * 8) return T;
  int t, tm, tn;
  if constexpr (LIST_ORDER) {
    // The 8 x 4 sub-blocks of all planes form one list (plane by plane, down the columns of sub-blocks); in a
    // round the eight XCDs take eight consecutive entries, i.e. neighbouring sub-blocks whose A' and B' panels
    // they share through the last-level cache.  g.chunk counts whole rounds of 32 tiles per XCD here.
    const int x = slot & 7, idx = slot >> 3;
    const int rnd = idx >> 5, within = idx & 31;
    const int sub_m = g.tiles_m >> 3, per_plane = sub_m * (g.tiles_n >> 2);
    const int entry = rnd * 8 + x;
    t = entry / g.div_plane;
    if (t >= g.num_moduli) return T;
    const int r = entry - t * per_plane;
    const int sn = r / g.div_rows, sm = r - sn * sub_m;
    tm = sm * 8 + (within & 7);
    tn = sn * 4 + (within >> 3);
  } else if (g.superblock) {
    // all eight XCDs work inside one 16 x 16 super-block of tiles at a time; XCD x owns the 8 x 4
    // sub-block (x & 1, x >> 1), so A' and B' panels missed by one L2 are found in the shared cache
    const int x = slot & 7, idx = slot >> 3;
    const int sb = idx >> 5, within = idx & 31;
    const int sbs_m = g.tiles_m >> 4, sbs_n = g.tiles_n >> 4;
    t = sb / g.div_plane;
    const int sr = sb - t * (sbs_m * sbs_n);
    // Structured products: the eight sub-blocks of a super-block hold different amounts of work (tiles beyond
    // the diagonal are skipped, tiles of a triangular operand differ in length), so the sub-block an XCD takes
    // rotates with the super-block and the modulus; over eight moduli every XCD has had every position.
    const int xp = (g.triangle | g.krange) ? ((x + sr + t) & 7) : x;
    // super-block coordinates; with a triangular operand the super-blocks with the longest tiles go first
    // (measured at 16384: 32.0 -> 30.1 ms for the product with a lower triangular first operand)
    const int by_rows = sr / g.div_rows, by_cols = sr / g.div_cols;
    int sm = sr - by_rows * sbs_m, sn = by_rows;
    if (g.krange == OZ2_KRANGE_UPTO_ROW) { sm = sbs_m - 1 - by_cols; sn = sr - by_cols * sbs_n; }
    if (g.krange == OZ2_KRANGE_FROM_ROW) { sm = by_cols; sn = sr - by_cols * sbs_n; }
    if (g.krange == OZ2_KRANGE_UPTO_COL) { sn = sbs_n - 1 - by_rows; }
    tm = sm * 16 + (xp & 1) * 8 + (within & 7);
    tn = sn * 16 + (xp >> 1) * 4 + (within >> 3);
    if (t >= g.num_moduli) return T;
  } else {
    const int item = (slot & 7) * g.chunk + (slot >> 3);
    if (item >= g.total) return T;
    const int per_t = g.tiles_m * g.tiles_n;
    t = item / g.div_plane;
    const int r = item - t * per_t;
    const int per_group = kGroupM * g.tiles_n;
    const int gid = r / g.div_group;
    const int first_m = gid * kGroupM;
    const int rr = r - gid * per_group;
    if (g.tiles_m - first_m < kGroupM) {
      tn = rr / g.div_last;
      tm = first_m + rr - tn * (g.tiles_m - first_m);
    } else {
      tn = rr / kGroupM;
      tm = first_m + rr % kGroupM;
    }
    if (g.folded != 0) unfold_triangle(g.folded, g.triangle, tm, tn);
  }
  // symmetric product: the other triangle of tiles is never needed
  if ((g.triangle == 1 && tm < tn) || (g.triangle == 2 && tm > tn)) return T;
  // Triangular operand (TRMM shape): op(A)(i, l) vanishes for l > i (lower) or l < i (upper), so the tile only
  // needs the k-tiles up to / from its diagonal block; which index (tm or tn) counts depends on the side.
  int kt_begin = 0, kt_end = g.ktiles;
  {
    const int per = BM / BK;  // k-tiles per diagonal block
    if (g.krange == OZ2_KRANGE_UPTO_ROW) kt_end = min(g.ktiles, (tm + 1) * per);
    if (g.krange == OZ2_KRANGE_FROM_ROW) kt_begin = min(g.ktiles, tm * per);
    if (g.krange == OZ2_KRANGE_UPTO_COL) kt_end = min(g.ktiles, (tn + 1) * per);
    if (g.krange == OZ2_KRANGE_FROM_COL) kt_begin = min(g.ktiles, tn * per);
  }
  const size_t kp = (size_t)g.k_pad;
  T.t = t;
  T.tm = tm;
  T.tn = tn;
  T.ktiles = kt_end - kt_begin;
  T.a_wave = g.a + ((size_t)t * g.m_pad + (size_t)tm * BM) * kp + wv * 64 * BK + (size_t)kt_begin * (BM * BK);
  T.b_wave = g.b + ((size_t)t * g.n_pad + (size_t)tn * BN) * kp + wv * 64 * BK + (size_t)kt_begin * (BN * BK);
  T.valid = true;
  return T;
}

// EARLY_ARRIVAL: a workgroup counts itself into the next round of the XCD synchronisation before its epilogue
// instead of after it (see the launcher).
// KBLOCKED: the inner dimension of a tile is walked in several k-blocks with a modular reduction of the
// accumulators between them (inner dimensions beyond the INT32 exactness bound, or a smaller block on request).
// A kernel of its own: the reduction's 256 x 8 instructions need so many registers at once that the compiler parks
// 48 accumulators in scratch memory around it, on the path of every tile, and the instantiation without it does not.
// SHORT: the inner dimension is at most OZ2_SHORT_SUM.  PASS_BY: residues are stored past the caches (see the launcher; as a branch around
// the stores it cost 1 to 2 % of the whole call).
template <bool RESIDUE_U8, bool LIST_ORDER, bool EARLY_ARRIVAL, bool KBLOCKED, bool SHORT = false, bool PASS_BY = false>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_num_vgpr(112))) gemm_i8_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char lds[];

  // stage 1 found an infinity or a NaN: the FP64 fallback forms C, these products would be thrown away
  if (g.skip_flag != nullptr && *g.skip_flag != 0ull) return;
  if (g.fin.slots != nullptr && blockIdx.x == 0) finish_scan(g.fin);

  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv >> 1, wn = wv & 1;

  // ---- which tiles: a workgroup takes the work indices blockIdx.x, blockIdx.x + gridDim.x, ...  With one
  // index per workgroup (gridDim.x = number of indices) this is a plain launch; with gridDim.x = number of
  // workgroup slots of the chip the loop keeps the launch order and lets the first copies of the next tile
  // fly while the current tile's epilogue runs.
  int slot = blockIdx.x;
  Tile cur = decode_tile<LIST_ORDER>(g, slot, wv);
  while (!cur.valid && slot < g.chunk * 8) {
    slot += gridDim.x;
    cur = decode_tile<LIST_ORDER>(g, slot, wv);
  }
  if (!cur.valid) return;

  // ---- global -> LDS copy: wave wv fills rows [64 wv, 64 wv + 64) of both tiles, 16 rows (1 KiB) per
  // load.  Lane l covers row (l >> 2) of the group and the chunk that the swizzle puts at position (l & 3).
  constexpr bool kSpreadRows = RESIDUE_U8;  // A' tiles of spread rows: the UINT8 epilogue's stores want them
  const unsigned voff = (unsigned)((lane >> 2) * BK) + (((lane & 3) ^ (lane >> 4)) << 4);
  unsigned voff_a[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) voff_a[q] = kSpreadRows ? (unsigned)((lane >> 2) * BK) + (((lane & 3) ^ q) << 4) : voff;
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds;
  const unsigned lds_wave = __builtin_amdgcn_readfirstlane(lds_base + wv * (64 * BK));

  // direct load q in 0..7 of a k-tile (pa, pb: this wave's first bytes of its A' and B' parts) into `stage`
  auto gl = [&](const int8_t* pa, const int8_t* pb, int stage, int q) {
    const unsigned sa = lds_wave + stage * kStageBytes;
    if (q < 4)
      load_to_lds_16(pa + q * 1024, voff_a[q & 3], sa + q * 1024);
    else
      load_to_lds_16(pb + (q - 4) * 1024, voff, sa + BM * BK + (q - 4) * 1024);
  };
  // k-tiles 0 .. NS-2 of a tile on their way into the stages from `base` on (the ring of stages runs on across tiles)
  // (a tile with fewer k-tiles fetches its k-tile 0 again in the place of those it lacks: every wait below can
  // then count on the same number of copies in flight)
  auto prologue_loads = [&](const Tile& T, int base) {
#pragma unroll
    for (int pth = 0; pth < NS - 1; ++pth) {
      const int st = base + pth >= NS ? base + pth - NS : base + pth;
      const int src = pth < T.ktiles ? pth : 0;
#pragma unroll
      for (int q = 0; q < kLoads; ++q) gl(T.a_wave + (size_t)src * (BM * BK), T.b_wave + (size_t)src * (BN * BK), st, q);
    }
  };

  // ---- LDS -> fragments: lane reads row (lane & 15) of a 16-row group, k-chunk lane / 16
  const int frag_off = (lane & 15) * BK + (((lane >> 4) ^ ((lane >> 2) & 3)) << 4);
  // (A' of spread rows: row 16 ((lane & 15) / 4) + 4 (x % 4) + lane % 4 of the 64, the same position within it)
  const int frag_off_a = kSpreadRows ? frag_off + (((lane & 12) << 2) + (lane & 3) - (lane & 15)) * BK : frag_off;
  const unsigned a_base = lds_base + wm * 128 * BK + frag_off_a, b_base = lds_base + BM * BK + wn * 128 * BK + frag_off;
  typedef const __attribute__((address_space(3))) v4i* LdsFrag;
  auto rd_a = [&](Frag& F, unsigned at, int x) { F.a[x] = *(LdsFrag)(at + (kSpreadRows ? (x & 4) * 16 + (x & 3) * 4 : x * 16) * BK); };
  auto rd_b = [&](Frag& F, unsigned at, int y) { F.b[y] = *(LdsFrag)(at + y * 16 * BK); };

  // Operand roles of v_mfma_i32_16x16x64_i8: the rows of the first operand run over the result registers
  // (lane l, register e: row 4 (l / 16) + e), the rows of the second over the lanes (row l % 16).
  //   UINT8 export: first = A', second = B': the four registers of a tile hold four consecutive rows i of one column, the four
  //   bytes of a word.
  //   INT32 export: first = B', second = A': a register holds sixteen consecutive rows i of each of four columns.
  // The 64 products of a k-tile: rows of tiles 0-3 against all eight columns, then rows 4-7; within a column back and forth, so
  // that every product shares an operand with the one before it.
  auto mfma = [&](const Frag& F, auto qc, auto first) {
    constexpr int q = decltype(qc)::value, y = (q >> 2) & 7, x = (q >> 5) * 4 + ((y & 1) ? 3 - (q & 3) : q & 3);
    const v4i& over_registers = RESIDUE_U8 ? F.a[x] : F.b[y];
    const v4i& over_lanes = RESIDUE_U8 ? F.b[y] : F.a[x];
    if constexpr (decltype(first)::value)
      Acc<8 * y + x>::template start<RESIDUE_U8>(over_registers, over_lanes);
    else
      Acc<8 * y + x>::add(over_registers, over_lanes);
  };

  named_accumulators();
  if (g.fin_stops) fetch_reports(g.fin, lds_base + (NS - 1) * kStageBytes, wv, lane);  // into the stage that the main loop fills first
  prologue_loads(cur, 0);
  if (g.fin_stops) {
    wait_vmcnt<(NS - 2) * kLoads>();
    __syncthreads();
    if (fetched_report_bad(g.fin, lds + (NS - 1) * kStageBytes)) {
      wait_vmcnt<0>();
      return;
    }
  }
  bool first = true;
  int round = 0;
  unsigned soff = 0;  // first byte of the stage that holds k-tile 0 of the current tile
  // One set of fragments: each is read again for the next k-tile after its last product and, two hundred cycles or more, before its
  // first one there.  Rows 4-7 and the last column of a k-tile arrive during its own first half.
  Frag F;
  const int xcd = blockIdx.x % kXcds;
  for (;;) {
  const int ktiles = cur.ktiles;
  const int t = cur.t, tm = cur.tm, tn = cur.tn;
  // ---- the next tile of this workgroup, if any.  Every iteration of the main loop below fetches one k-tile, NS - 1
  // ahead of the one it multiplies.  When that runs past the end of this tile and both tiles are at least NS - 1
  // k-tiles long, it fetches the first k-tiles of the next tile: its copies then cost no time of their own at the
  // tile boundary.  Otherwise the slot fetches this tile's k-tile 0 once more into a stage nobody reads again (one
  // loop body for every iteration, the same number of copies in flight at every wait).
  Tile nxt;
  nxt.valid = false;
  do {
    slot += gridDim.x;
    nxt = decode_tile<LIST_ORDER>(g, slot, wv);
  } while (!nxt.valid && slot < g.chunk * 8);
  const bool across = nxt.valid && ktiles >= NS - 1 && nxt.ktiles >= NS - 1;
  const int8_t* const over_a = across ? nxt.a_wave : cur.a_wave;
  const int8_t* const over_b = across ? nxt.b_wave : cur.b_wave;

  // ---- k-tiles 0 .. NS-2 are in flight: make tile 0 visible, its first fragments in registers.  After the first
  // tile of the loop the kStores stores of the previous epilogue were issued behind those copies; the counter goes
  // down in issue order, so a wait that leaves that many more operations outstanding covers the copies alone and the
  // stores drain during the first k-tiles.
  if (first)
    wait_vmcnt<(NS - 2) * kLoads>();
  else
    wait_vmcnt<(NS - 2) * kLoads + kStores>();
  if (g.xcd_sync != nullptr && round < g.full_rounds && threadIdx.x == 0) {
    // The workgroups of an XCD start their tiles of a round together.  The wait is bounded (about a millisecond).
    // If it runs to its bound, the workgroups of this XCD are not all resident at once (another kernel holds
    // compute units) or the counters were not cleared: the counter is then pushed beyond every target of this
    // launch, so that no workgroup of the XCD waits again -- the launch loses one bound, not one per round.
    // (A flag kept in a register instead would live across the main loop, where no register is free.)
    unsigned long long* c = g.xcd_sync + xcd;
    if (!EARLY_ARRIVAL || round == 0) atomicAdd(c, 1ull);
    const unsigned long long target = (unsigned long long)(gridDim.x / kXcds) * (unsigned long long)(round + 1);
    bool arrived = false;
    for (int spins = 0; spins < g.sync_spins; ++spins) {
      if (__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target) {
        arrived = true;
        break;
      }
      __builtin_amdgcn_s_sleep(8);
    }
    if (!arrived) {
      atomicAdd(c, 1ull << 40);
      wait_vmcnt<0>();
    }
  }
  ++round;
  const int store_window = first ? 0 : NS - 2;
  first = false;
  unsigned ra = a_base + soff, rb = b_base + soff;  // where this lane's fragments of the current k-tile start
  __syncthreads();
#pragma unroll
  for (int x = 0; x < 4; ++x) rd_a(F, ra, x);
#pragma unroll
  for (int y = 0; y < 7; ++y) rd_b(F, rb, y);

  // fa, fb: where the next fetch reads (k-tile kt + NS - 1 of this tile while that exists), and its step from k-tile to k-tile
  const int8_t* fa = NS - 1 < ktiles ? cur.a_wave + (size_t)(NS - 1) * (BM * BK) : cur.a_wave;
  const int8_t* fb = NS - 1 < ktiles ? cur.b_wave + (size_t)(NS - 1) * (BN * BK) : cur.b_wave;
  const unsigned over_step = across ? BM * BK : 0;
  unsigned fstep = NS - 1 < ktiles ? BM * BK : over_step;
  // k-tile kt: its products; the fragments of k-tile kt + 1; the loads of k-tile kt + NS - 1.  A product takes the matrix core 16
  // cycles and every other instruction four or five of issue, so that not more than two stand between products.
  auto ktile = [&](int kt, auto first) {
    unsigned noff, na, nb, fill;
    unrolled<64>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      mfma(F, qc, first);
      if constexpr (q == 1) rd_b(F, rb, 7);
      if constexpr (q >= 4 && q < 20 && q % 4 == 0) rd_a(F, ra, 4 + (q - 4) / 4);
      // (each statement pinned to its place: the compiler would collect them in one)
      if constexpr (q == 18) {
        noff = (soff + kStageBytes) & (kLdsBytes - 1);
        asm volatile("" : "+s"(noff));
      }
      if constexpr (q == 20) {
        na = a_base + noff;
        asm volatile("" : "+v"(na));
      }
      if constexpr (q == 21) {
        nb = b_base + noff;
        asm volatile("" : "+v"(nb));
      }
      if constexpr (q == 23) {
        fill = lds_wave + ((soff + (NS - 1) * kStageBytes) & (kLdsBytes - 1));  // k-tile kt - 1's stage
        asm volatile("" : "+s"(fill));
      }
      // from k-tile ktiles - NS + 1 on the fetches run past the end of this tile
      if constexpr (q == 25) {
        fa = kt + NS - 1 == ktiles ? over_a : fa;
        asm volatile("" : "+s"(fa));
      }
      if constexpr (q == 27) {
        fb = kt + NS - 1 == ktiles ? over_b : fb;
        asm volatile("" : "+s"(fb));
      }
      if constexpr (q == 29) {
        fstep = kt + NS - 1 == ktiles ? over_step : fstep;
        asm volatile("" : "+s"(fstep));
      }
      if constexpr (q == kSyncAt) {
        // k-tile kt+1 must be complete in LDS for every wave before anyone reads it; passing this barrier
        // also means every wave has finished reading k-tile kt-1, whose stage is refilled below.  In the first NS - 2
        // iterations the previous epilogue's stores lie between the copies waited for and the newest operation.
        wait_vmcnt_unless_below<(NS - 3) * kLoads, (NS - 3) * kLoads + kStores>(kt, store_window);
        __syncthreads();
      }
      // rows of the next k-tile's first half, then its columns (c is used for the last time at product 35 + 4 c)
      if constexpr (q == 35) rd_a(F, na, 0);
      if constexpr (q == 37) rd_a(F, na, 1);
      if constexpr (q == 40) rd_a(F, na, 2);
      if constexpr (q == 43) rd_a(F, na, 3);
      if constexpr (q == 44) rd_b(F, nb, 0);
      if constexpr (q == 47) rd_b(F, nb, 1);
      if constexpr (q == 50) rd_b(F, nb, 2);
      if constexpr (q == 53) rd_b(F, nb, 3);
      if constexpr (q == 55) rd_b(F, nb, 4);
      if constexpr (q == 58) rd_b(F, nb, 5);
      if constexpr (q == 60) rd_b(F, nb, 6);
      if constexpr (q == 34) set_lds_target(fill);
      if constexpr (q == 46) set_lds_target(fill + BM * BK);
      if constexpr (q >= 36 && q <= 45 && q % 3 == 0) load_to_lds_target<(q - 36) / 3 * 1024>(fa, voff_a[(q - 36) / 3]);
      if constexpr (q >= 48 && q <= 57 && q % 3 == 0) load_to_lds_target<(q - 48) / 3 * 1024>(fb, voff);
      if constexpr (q == 61) fa += fstep;
      if constexpr (q == 62) fb += fstep;
      if constexpr (q == 63) {
        soff = noff;
        ra = na;
        rb = nb;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  const Oz2FoldConsts& fc = g.fold[t / g.per_modulus];
  const Oz2FoldConsts fv = in_vector_registers(fc);  // ahead of the main loop, which hides their loads
  // The first products of a tile start from an inline constant of the instruction (clearing 256 accumulators takes
  // 8 cycles each, 2000 of the tile's 30000 at k = 1024), so k-tile 0 stands before the loop.
  ktile(0, std::true_type());
  int block_end = KBLOCKED ? g.ktiles_per_block : 0;
  // Where the loop starts: the same instructions take up to 1 % longer at other places (first statement behind a multiple of 64, four
  // bytes each: 0 / 4 / 8 / 12 instructions, 16384^3 51.76 / 51.23 / 51.67 / 51.20 ms, 4096^3 1084 / 1071 / 1078 / 1073 us).
  asm volatile(
      ".p2align 6\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop "
      "0\n\ts_nop 0");
  for (int kt = 1; kt < ktiles; ++kt) {
    if constexpr (KBLOCKED) {
      if (kt == block_end) {  // between k-blocks: bring the accumulators back near zero
        block_end += g.ktiles_per_block;
        settle_acc();
        unrolled<64>([&](auto tile) {
          constexpr int T = decltype(tile)::value;
          constexpr int start = RESIDUE_U8 ? (int)OZ2_ACC_START : 0;
          unrolled<4>([&](auto e) {
            Acc<T>::write(decltype(e)::value, (unsigned)(reduce_mod((int)Acc<T>::read(decltype(e)::value) - start, fc.p, fc.inv_p) + start));
          });
        });
        settle_acc();
      }
    }
    ktile(kt, std::false_type());
  }

  // ---- a next tile whose first copies were not fetched by the main loop above: they fly during the epilogue
  // below.  The barrier makes sure that every wave has left the main loop (all LDS reads of this tile issued) before
  // stages refill.  `soff` is by now the stage after this tile's last k-tile, where the next tile starts.
  if (nxt.valid) {
    if (!across) {
      __syncthreads();
      prologue_loads(nxt, (int)(soff / kStageBytes));
    }
    if constexpr (EARLY_ARRIVAL) {
      // count in for the next round now: the others then wait for this workgroup's main loop only, not for its
      // epilogue, and the counter's round trip overlaps the epilogue
      if (g.xcd_sync != nullptr && round < g.full_rounds && threadIdx.x == 0)
        atomicAdd(g.xcd_sync + xcd, 1ull);
    }
  }

  // ---- epilogue
  settle_acc();
  // Sixteen residues of column y of MFMA tiles, those of tiles 4 h .. 4 h + 3: rows 16 (lane / 16) + (0..15) of 64, column lane % 16, one
  // byte each.
  auto residues = [&](auto yc, auto hc) {
    constexpr int T = 8 * decltype(yc)::value + 4 * decltype(hc)::value;
    unsigned v[16], w[4];
    if constexpr (SHORT) {
      unrolled<4>([&](auto xc) { Acc<T + decltype(xc)::value>::low_words(v + 4 * decltype(xc)::value, fv.recip, fv.half); });
#pragma unroll
      for (int x = 0; x < 4; ++x) w[x] = oz2_short_residues4(v + 4 * x, (unsigned)fv.p);
    } else {
      // (step by step: a byte dot product's result can only be read three instructions later)
      unrolled<16>([&](auto e) { v[e] = Acc<T + e / 4>::fold_sum(decltype(e)::value % 4, fv.kpack, fv.base); });
      settle_sums(v);
#pragma unroll
      for (int x = 0; x < 4; ++x) w[x] = oz2_fold_residues4(v + 4 * x, fv);
    }
    __builtin_amdgcn_sched_barrier(0);
    return v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
  };
  if (RESIDUE_U8) {
    // Algorithm 1 line 7 here: c'' = c' mod p in [0, p), four residues per 32-bit word.  Lane holds column
    // j = lane % 16 of an MFMA tile, its four registers four consecutive rows i, those of four tiles sixteen.
    // Bound by instruction issue, one wave per SIMD: 3.25 instructions of 5 cycles per element, and the 8-cycle move for
    // the half that sits in accumulation registers (before: seven, the move for all, and 2000 cycles to clear the
    // accumulators for the next tile).  With the stores left to drain and the tile decoding on the scalar unit the
    // work between two main loops went from 13000 to 7500 cycles: GEMM of 18 moduli at 8192 x 8192 x 1024 1.31 -> 1.20 ms
    // (2.08 POP/s), of 16 at 4096^3 0.87 -> 0.85, of 14 at 2048^3 0.115 -> 0.108, of 26 at 8192^3 10.67 -> 10.50.
    // the wave's corner of the tile (uniform over the wave) and the lane's own offset from it (column lane % 16,
    // rows 16 (lane / 16) ..: below 2^32, m_pad is below 2^27)
    uint8_t* const corner = reinterpret_cast<uint8_t*>(g.c) + (size_t)t * g.n_pad * g.m_pad +
                            ((size_t)tn * BN + wn * 128) * g.m_pad + (size_t)tm * BM + wm * 128;
    // (formed again for every tile from the lane number as the hardware counts it: a value kept across the main
    // loop, where no register is free, would be parked in scratch memory and fetched per tile)
    unsigned start = 0u;
    asm volatile("" : "+s"(start));  // opaque zero: the count below is taken here, in every tile
    const unsigned lane_now = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, start));
    const unsigned lane_off = (lane_now & 15u) * (unsigned)g.m_pad + 16u * (lane_now >> 4);
    unrolled<8>([&](auto yc) {
      constexpr int y = decltype(yc)::value;
      const v4i lo = residues(yc, std::integral_constant<int, 0>()), hi = residues(yc, std::integral_constant<int, 1>());
      // both halves of a column together, so that its cache lines are complete at once
      uint8_t* cj = corner + (size_t)(y * 16) * g.m_pad;  // uniform; + 64 h + lane_off below
      v4i* const to = reinterpret_cast<v4i*>(cj + lane_off);
      if constexpr (PASS_BY) {
        __builtin_nontemporal_store(lo, to);
        __builtin_nontemporal_store(hi, to + 4);
      } else {
        to[0] = lo;
        to[4] = hi;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  } else {
    // Register e of tile (x, y) holds rows 16 x + lane % 16 of column 16 y + 4 (lane / 16) + e.  Exchanged between the groups of
    // sixteen lanes of two tiles, a register has 32 consecutive rows of two columns: every store fills two cache lines.  (16 bytes
    // per lane, 64 bytes of each of sixteen columns, meet in the same channels where the columns are a power of two apart: whole calls
    // with 16 moduli, us, 8192 x 8192 x 1024 2610 -> 2412, 4096^3 1298 -> 1280, INT8-product mode 500^3 58.5 -> 54.4.)
    int* plane = g.c + ((size_t)t * g.n_pad + (size_t)tn * BN + wn * 128 + 8 * (lane >> 5)) * g.m_pad + (size_t)tm * BM + wm * 128 + (lane & 31);
    unrolled<8>([&](auto yc) {
      unrolled<4>([&](auto xc) {
        unrolled<4>([&](auto ec) {
          constexpr int x = 2 * decltype(xc)::value, y = decltype(yc)::value, e = decltype(ec)::value;
          const auto s = __builtin_amdgcn_permlane16_swap(Acc<8 * y + x>::read(e), Acc<8 * y + x + 1>::read(e), false, false);
          int* p = plane + (size_t)(y * 16 + e) * g.m_pad + x * 16;
          p[0] = (int)s[0];
          p[4 * g.m_pad] = (int)s[1];
        });
      });
    });
  }
  if (!nxt.valid) {
    wait_vmcnt<0>();  // the copies fetched beyond the end of the last tile must have landed before the LDS is given back
    break;
  }
  cur = nxt;
  }  // loop over this workgroup's tiles
}

__global__ void clear_sync_kernel(unsigned long long* counters, int count) {
  if ((int)threadIdx.x < count) counters[threadIdx.x] = 0ull;
}

}  // namespace

namespace {

// Once per process: the kernels' dynamic LDS limit and the number of compute units (a multiple of 8, one
// workgroup slot each).  Callers hold the library's lock.
int g_cus = 0;
int g_sync_spins = 4096;  // polls per wait of the round synchronisation (each followed by a short sleep); 0: off
constexpr Oz2ScanFinish kNothing = {nullptr, 0u, nullptr, 0};
hipError_t gemm_setup() {
  if (g_cus) return hipSuccess;
#define OZ2_BOTH(U8, LIST, EARLY)                                              \
  reinterpret_cast<const void*>(gemm_i8_kernel<U8, LIST, EARLY, false>),       \
      reinterpret_cast<const void*>(gemm_i8_kernel<U8, LIST, EARLY, true>)
#define OZ2_SHALLOW(SHORT, PASS_BY)                                                           \
  reinterpret_cast<const void*>(gemm_i8_kernel<true, false, false, false, SHORT, PASS_BY>),   \
      reinterpret_cast<const void*>(gemm_i8_kernel<true, true, false, false, SHORT, PASS_BY>)
  const void* kernels[18] = {OZ2_SHALLOW(true, false), OZ2_SHALLOW(true, true), OZ2_SHALLOW(false, true),
                             OZ2_BOTH(false, false, false), OZ2_BOTH(true, false, false), OZ2_BOTH(false, true, false),
                             OZ2_BOTH(true, true, false),   OZ2_BOTH(true, false, true),  OZ2_BOTH(true, true, true)};
#undef OZ2_BOTH
#undef OZ2_SHALLOW
  hipError_t e = hipSuccess;
  for (int i = 0; i < 18 && e == hipSuccess; ++i)
    e = hipFuncSetAttribute(kernels[i], hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
  if (e != hipSuccess) return e;
  int dev = 0, n = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  g_cus = n / 8 * 8 < 8 ? 8 : n / 8 * 8;
  return hipSuccess;
}

// num_moduli planes of A' (off_a) times planes of B' (off_b) -> planes of C' (off_c); plane t is reduced
// b_is_a: the second operand's planes are the first operand's (symmetric product; m_pad == n_pad)
// (moduli: one per per_modulus consecutive planes)
hipError_t launch_gemm(const Oz2Layout& lay, char* ws, int num_moduli, const int* moduli, int per_modulus, int64_t kblock,
                       int residue_u8, int triangle, int krange, bool b_is_a, bool check_flag, const Oz2ScanFinish& fin,
                       hipStream_t st) {
  hipError_t e = gemm_setup();
  if (e != hipSuccess) return e;
  if (num_moduli < 1 || num_moduli > OZ2_MAX_PLANES) return hipErrorInvalidValue;
  GemmArgs g;
  g.a = reinterpret_cast<const int8_t*>(ws + lay.off_a);
  g.b = reinterpret_cast<const int8_t*>(ws + (b_is_a ? lay.off_a : lay.off_b));
  if (b_is_a && lay.m_pad != lay.n_pad) return hipErrorInvalidValue;
  g.triangle = triangle;
  g.krange = krange;
  // (with reports still to be turned into the flag by this launch, nobody can look at the flag yet)
  g.skip_flag = check_flag && !fin.slots ? reinterpret_cast<const unsigned long long*>(ws + lay.off_flags) : nullptr;
  g.fin = fin;
  g.fin_stops = 0;
  g.c = reinterpret_cast<int*>(ws + lay.off_c);
  g.m_pad = lay.m_pad;
  g.n_pad = lay.n_pad;
  g.k_pad = lay.k_pad;
  if (lay.m_pad >= ((int64_t)1 << 27)) return hipErrorInvalidValue;  // the epilogue's lane offsets: 15 m_pad + 48 in 32 bits
  g.tiles_m = (int)(lay.m_pad / BM);
  g.tiles_n = (int)(lay.n_pad / BN);
  g.num_moduli = num_moduli;
  g.superblock = (g.tiles_m % 16 == 0 && g.tiles_n % 16 == 0) ? 1 : 0;
  // Symmetric product outside the super-block order: only the tiles of the triangle are counted, so that they are launched
  // like those of a general product, one workgroup per compute unit (16 moduli, inner dimension 1024, whole calls: dsyrk of
  // order 5000 425 -> 393 us, of order 10000 1447 -> 1333).
  g.folded = triangle != 0 && !g.superblock ? g.tiles_m : 0;
  if (g.folded) fold_triangle(g.folded, &g.tiles_m, &g.tiles_n);
  const int64_t total = (int64_t)g.tiles_m * g.tiles_n * num_moduli;
  if (total > (int64_t)1 << 30) return hipErrorInvalidValue;
  g.total = (int)total;
  g.chunk = (int)((total + 7) / 8);
  // list order of the 8 x 4 sub-blocks: general products whose tile grid is a multiple of 8 x 4 but not of 16 x 16
  // (and at least eight rounds of them: with a handful of sub-blocks the range order spreads the tiles better)
  const bool list_order = !g.superblock && triangle == 0 && krange == OZ2_KRANGE_ALL && g.tiles_m % 8 == 0 &&
                          g.tiles_n % 4 == 0 && total / 32 >= 64;
  if (list_order) g.chunk = (int)((total / 32 + 7) / 8) * 32;  // whole rounds of 32 tiles per XCD
  if (list_order) {
    g.div_rows = fast_div((unsigned)(g.tiles_m / 8));
    g.div_plane = fast_div((unsigned)(g.tiles_m / 8 * (g.tiles_n / 4)));
  } else if (g.superblock) {
    g.div_rows = fast_div((unsigned)(g.tiles_m / 16));
    g.div_plane = fast_div((unsigned)(g.tiles_m / 16 * (g.tiles_n / 16)));
  } else {
    g.div_rows = fast_div(1);
    g.div_plane = fast_div((unsigned)(g.tiles_m * g.tiles_n));
  }
  g.div_cols = fast_div((unsigned)(g.superblock ? g.tiles_n / 16 : 1));
  g.div_group = fast_div((unsigned)(kGroupM * g.tiles_n));
  g.div_last = fast_div((unsigned)(g.tiles_m % kGroupM ? g.tiles_m % kGroupM : 1));
  g.ktiles = (int)(lay.k_pad / BK);
  // (UINT8: a little below what INT32 holds, see OZ2_ACC_START; the residues do not depend on the blocks)
  g.ktiles_per_block = (int)((residue_u8 && kblock > OZ2_ACC_BLOCK ? OZ2_ACC_BLOCK : kblock) / BK);
  g.per_modulus = fast_div((unsigned)per_modulus);
  for (int t = 0; t < num_moduli / per_modulus; ++t) g.fold[t] = oz2_fold_consts(moduli[t]);
  // General products: one workgroup per compute unit (each holds one: 128 KiB of LDS, 512 registers per lane),
  // every workgroup walks the work indices of its slot in launch order.  Structured products have tiles of
  // unequal length (or none): there the hardware's dynamic placement of one workgroup per index balances better.
  unsigned grid = (unsigned)(g.chunk * 8);
  g.xcd_sync = nullptr;
  g.full_rounds = 0;
  g.sync_spins = g_sync_spins;
  if ((triangle == 0 || g.folded) && krange == OZ2_KRANGE_ALL) {
    if (grid > (unsigned)g_cus) grid = (unsigned)g_cus;
    // General products: the workgroups of an XCD start the tiles of a round together, which keeps them
    // on the same k-tiles of their shared panels (measured: L2 misses 48.7 GiB per launch every time instead of
    // 50-54 GiB, and 83 GiB in some runs).  The counters are words 8..15 of the flag words that stage 1 clears.
    // Only for inner dimensions above 6144: shorter panels stay in the L2 anyway and the wait for the slowest
    // workgroup of every round costs more than it saves (measured without it: -10 % at k = 1024, -6 % at 2048,
    // -4 % at 4096, -3 % at 6144, -1.5 % at 8192 with 64 rounds but +1 % at 8192 with 448 rounds).
    if (num_moduli > 1 && g.ktiles > 96 && g_sync_spins > 0) {
      g.xcd_sync = reinterpret_cast<unsigned long long*>(ws + lay.off_flags) + 8;
      // rounds in which each of the grid / 8 workgroup slots of every XCD has a tile: all of them in the
      // super-block order (its work count is a multiple of 256); otherwise XCD 7 runs out first
      const int per_xcd = (int)grid / 8;
      const int last = g.total - 7 * g.chunk;  // work items of XCD 7
      g.full_rounds = g.superblock ? (g.chunk * 8) / (int)grid : (last > 0 ? last / per_xcd : 0);
      // list order: the rounds in which all eight XCDs have a sub-block, when a round of the launch (32 workgroups
      // per XCD) is a round of the list
      if (list_order) g.full_rounds = per_xcd == 32 ? (int)(total / 256) : 0;
    }
  }
  // Early arrival at the round synchronisation: with tiles of up to 128 k-tiles (measured at 8192: -1 % of the
  // GEMM time with 448 rounds, -1.5 % with 64); with longer tiles the tighter form keeps the workgroups closer
  // together on their panels and is the faster one.  UINT8 epilogue only.
  const bool early = residue_u8 && g.xcd_sync != nullptr && g.ktiles <= 128;
  // Stage 1 left the flag to this launch and non-finite inputs do not need these products (1.2 ms of 9 at 8192 x 8192 x 1024
  // with 16 moduli).  A launch whose workgroups walk five tiles or more has each of them look at the reports first (16 moduli,
  // finite inputs, whole calls with / without it, us: dsyrk of order 5000 378 / 376, 4096 x 4096 x 1024 440 / 440), but not
  // more than 4096 of them; with one workgroup per tile (dtrmm 1024 x 16384 527 / 511) or more reports than that the flag word
  // is formed ahead of the launch.
  if (check_flag && fin.slots) {
    const int64_t each = 720 * (krange == OZ2_KRANGE_ALL ? g.ktiles : (g.ktiles + 1) / 2) + 4500;
    const bool wait = (triangle && !g.folded ? total / 2 : total) / g_cus * each >= OZ2_FINISH_FIRST_NS;
    if (((grid <= (unsigned)g_cus && total > 4 * (int64_t)g_cus) || (fin.stops && !wait)) && fin.count <= kStageBytes / 8) {
      g.fin_stops = 1;
    } else if (wait || fin.stops) {
      if ((e = oz2_launch_finish_scan(fin, st)) != hipSuccess) return e;
      g.fin = kNothing;
      g.skip_flag = reinterpret_cast<const unsigned long long*>(ws + lay.off_flags);
    }
  }
  // The round synchronisation needs its counters cleared before the launch, which comes with forming the flag word.
  if (g.xcd_sync != nullptr && g.fin.slots) {
    if ((e = oz2_launch_finish_scan(fin, st)) != hipSuccess) return e;
    g.fin = kNothing;
    g.fin_stops = 0;
    if (check_flag) g.skip_flag = reinterpret_cast<const unsigned long long*>(ws + lay.off_flags);
  }
  const dim3 grd(grid), thr(kThreads);
  // tiles walked in one k-block (the usual case) take the instantiation without the reduction between k-blocks
  const bool kblocked = g.ktiles_per_block < g.ktiles;
#define OZ2_GEMM(U8, LIST, EARLY)                                                                   \
  do {                                                                                              \
    if (kblocked)                                                                                   \
      hipLaunchKernelGGL((gemm_i8_kernel<U8, LIST, EARLY, true>), grd, thr, kLdsBytes, st, g);      \
    else                                                                                            \
      hipLaunchKernelGGL((gemm_i8_kernel<U8, LIST, EARLY, false>), grd, thr, kLdsBytes, st, g);     \
  } while (0)
  // Inner dimensions up to 2048: no round synchronisation, and residues stored past the caches.  Where the panels of a round of tiles are
  // of the L2's size, the lines of C' push them out and the copies into LDS wait (cycles per k-tile at 8192 x 8192 x 1024 1510 -> 1240,
  // inside the kernel).  Not where the last-level cache keeps them for stage 3, but for results that the L2s hold whole, which they
  // would give back at the end of the launch, one line after the other.  Whole calls, us, through / past: 12 moduli 8000 x 4000 x 300 381
  // / 337, 16 moduli 4000 x 4000 x 600 316 / 292, 18 moduli 8192 x 8192 x 1024 1629 / 1572, 16 moduli 8192 x 8192 x 2048 2210 / 2169, 14
  // moduli 1024^3 38.2 / 36.9; 2000 x 2000 x 500 71.8 / 75.8, 2048^3 171.1 / 172.1, 15 moduli 3001 x 2777 x 1000 194 / 198; longer ones:
  // 14 moduli 4000 x 4000 x 2400 611 / 613, 16 moduli 6000 x 6000 x 3000 1692 / 1698, 2048 x 2048 x 8192 616 / 622, 8192^3 7042 / 7076.
  const int64_t result = total * (BM * BN);
  const bool shallow = residue_u8 && !kblocked && g.ktiles <= 32 && g.xcd_sync == nullptr;
  const bool short_sums = lay.k_pad <= OZ2_SHORT_SUM, pass_by = result > OZ2_CACHED_RESULT || result <= (int64_t)1 << 25;
#define OZ2_GEMM_SHALLOW(SHORT, PASS_BY)                                                                            \
  do {                                                                                                              \
    if (list_order)                                                                                                 \
      hipLaunchKernelGGL((gemm_i8_kernel<true, true, false, false, SHORT, PASS_BY>), grd, thr, kLdsBytes, st, g);   \
    else                                                                                                            \
      hipLaunchKernelGGL((gemm_i8_kernel<true, false, false, false, SHORT, PASS_BY>), grd, thr, kLdsBytes, st, g);  \
  } while (0)
  if (shallow && short_sums && pass_by)
    OZ2_GEMM_SHALLOW(true, true);
  else if (shallow && short_sums)
    OZ2_GEMM_SHALLOW(true, false);
  else if (shallow && pass_by)
    OZ2_GEMM_SHALLOW(false, true);
  else if (!residue_u8 && list_order)
    OZ2_GEMM(false, true, false);
  else if (!residue_u8)
    OZ2_GEMM(false, false, false);
  else if (list_order && early)
    OZ2_GEMM(true, true, true);
  else if (list_order)
    OZ2_GEMM(true, true, false);
  else if (early)
    OZ2_GEMM(true, false, true);
  else
    OZ2_GEMM(true, false, false);
#undef OZ2_GEMM
#undef OZ2_GEMM_SHALLOW
  return hipGetLastError();
}

}  // namespace

hipError_t oz2_gemm_setup() { return gemm_setup(); }

int oz2_gemm_cus() { return g_cus; }

void oz2_gemm_set_sync_spins(int spins) { g_sync_spins = spins; }

// The round synchronisation counts on counters that are zero at launch.  Stage 1 clears them with the row
// maxima; a GEMM launched without a stage 1 before it (the staged entry point called again) clears them here.
hipError_t oz2_launch_clear_sync(const Oz2Layout& lay, char* ws, hipStream_t st) {
  hipLaunchKernelGGL(clear_sync_kernel, dim3(1), dim3(64), 0, st,
                     reinterpret_cast<unsigned long long*>(ws + lay.off_flags) + 8, kXcds);
  return hipGetLastError();
}

hipError_t oz2_launch_stage2(const Oz2Plan& plan, const Oz2Layout& lay, char* ws, int64_t kblock, int residue_u8,
                             int triangle, int krange, int check_flag, const Oz2ScanFinish& fin, hipStream_t st) {
  return launch_gemm(lay, ws, plan.N, plan.moduli, 1, kblock, residue_u8, triangle, krange, triangle != 0, check_flag != 0, fin,
                     st);
}

// The seven products per modulus of the Strassen form: 7 N planes of half the extents of lay, plane 7 t + s
// reduced modulo p_t in the epilogue (UINT8 residues).
hipError_t oz2_launch_strassen_gemm(const Oz2Plan& plan, const Oz2Layout& lay, char* ws, int64_t kblock, int check_flag,
                                    hipStream_t st) {
  Oz2Layout half = lay;
  half.m_pad = lay.m_pad / 2;
  half.n_pad = lay.n_pad / 2;
  half.k_pad = lay.k_pad / 2;
  if (half.m_pad % BM || half.n_pad % BN || half.k_pad % BK) return hipErrorInvalidValue;
  return launch_gemm(half, ws, 7 * plan.N, plan.moduli, 7, kblock, 1, 0, OZ2_KRANGE_ALL, false, check_flag != 0, kNothing, st);
}

// One plain INT8 product with INT32 output and no modular reduction between k-blocks: the caller guarantees
// k_pad * 64 * 64 < 2^31.
hipError_t oz2_launch_bound_gemm(const Oz2Layout& lay, char* ws, bool symmetric, hipStream_t st) {
  const int one = 1;
  return launch_gemm(lay, ws, 1, &one, 1, lay.k_pad, 0, 0, OZ2_KRANGE_ALL, symmetric, false, kNothing, st);
}
