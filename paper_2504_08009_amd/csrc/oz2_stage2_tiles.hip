// Stage 2 for small products (Algorithm 1 lines 6-7, UINT8 residues): the same operand planes, MFMA instruction, LDS
// layout and residue arithmetic as gemm_i8_kernel (oz2_stage2.hip), with tiles of 128 x 128 or 64 x 64 and several
// workgroups per compute unit in the place of one persistent workgroup with a 256 x 256 tile.
//
// A product of a few 256 x 256 tiles per modulus leaves most of the chip idle (14 workgroups for 256 x 256 x 256 with 14
// moduli) and computes the padding of its last tiles (60 % of the work at 333 x 517); the time is that of one tile from
// launch to last store.  Smaller tiles cost more L2 -> LDS bytes per operation (twice as many at 128 x 128, four times at
// 64 x 64) but there is bandwidth to spare at these sizes, and rows and columns beyond the matrices are not touched.
// Which sizes come here, with both sides' times: tile_size below.
//
// One workgroup of four waves (2 x 2) per tile, the k-tiles of 64 bytes in a ring of NS LDS stages filled by direct
// loads NS - 1 ahead; the other workgroups of the compute unit work while one waits for its first copies or stores its
// residues.  256 registers per lane or less: the accumulators are ordinary registers (build.py builds this file with
// -amdgpu-mfma-vgpr-form), so the epilogue reads them directly.
#include "oz2_bound.h"
#include "oz2_gemm.h"
#include "oz2_scan_finish.h"
#include "oz2_warm.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int BK = OZ2_TILE_K;
constexpr int kThreads = 256;
constexpr int kBlk = OZ2_TILE_M;  // rows of a block of the plane layout
static_assert(OZ2_TILE_M == 256 && OZ2_TILE_N == 256 && OZ2_TILE_K == 64, "plane layout is 256 x 64 blocks");
constexpr int kGroup = 8;         // tile rows of a column group

struct TileArgs {
  const int8_t* a;
  const int8_t* b;
  uint8_t* c;
  int64_t m_pad, n_pad, k_pad;
  int tiles_m, tiles_n, total, chunk;  // tiles, and tiles per die
  int ktiles, triangle, folded, krange;  // as in the large kernel
  const unsigned long long* skip_flag;
  Oz2ScanFinish fin;
  int fin_stops;  // 1: every workgroup looks at the reports and stops when one is bad
  FastDiv div_plane, div_group, div_last;
  Oz2FoldConsts fold[OZ2_MAX_N];
};

// MI x NI MFMA tiles of 32 x 32 per wave, NS stages, WGS workgroups per compute unit; WARM: a launch of few workgroups
// MAXIMA: the one product of the bound planes of the INT8-product mode (Section 4.1).  Only its row and column maxima are wanted: they
// are gathered here (c holds the words of the rows, then those of the columns, zero before the launch; the rows' for both where the
// product is symmetric), and the INT32 product, 4 bytes an element written and read again, does not exist.
template <int MI, int NI, int NS, int WGS, bool WARM, bool MAXIMA>
__global__ void __launch_bounds__(kThreads, WGS) gemm_i8_tile_kernel(const TileArgs g) {
  constexpr int TM = 64 * MI, TN = 64 * NI;
  constexpr int kStage = (TM + TN) * BK;
  constexpr int kLoadsA = MI, kLoadsB = NI, kLoads = kLoadsA + kLoadsB;  // direct loads of 1 KiB per wave and k-tile
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  if constexpr (WARM && !MAXIMA) warm_arguments(g);

  if (g.skip_flag != nullptr && *g.skip_flag != 0ull) return;
  if (g.fin.slots != nullptr && !g.fin_stops && blockIdx.x == 0) finish_scan(g.fin);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv >> 1, wn = wv & 1;

  // workgroup i of a launch runs on die i % 8: each die takes a contiguous range of tiles, in column groups of kGroup rows
  const int item = (int)(blockIdx.x & 7) * g.chunk + (int)(blockIdx.x >> 3);
  if (item >= g.total) return;
  const int t = item / g.div_plane;
  const int r = item - t * (g.tiles_m * g.tiles_n);
  const int gid = r / g.div_group;
  const int first_m = gid * kGroup, rr = r - gid * (kGroup * g.tiles_n);
  int tm, tn;
  if (g.tiles_m - first_m < kGroup) {
    tn = rr / g.div_last;
    tm = first_m + rr - tn * (g.tiles_m - first_m);
  } else {
    tn = rr / kGroup;
    tm = first_m + rr % kGroup;
  }
  if (g.folded != 0) unfold_triangle(g.folded, g.triangle, tm, tn);
  int kt_begin = 0, kt_end = g.ktiles;
  if (g.krange == OZ2_KRANGE_UPTO_ROW) kt_end = min(g.ktiles, (tm + 1) * (TM / BK));
  if (g.krange == OZ2_KRANGE_FROM_ROW) kt_begin = tm * (TM / BK);
  if (g.krange == OZ2_KRANGE_UPTO_COL) kt_end = min(g.ktiles, (tn + 1) * (TN / BK));
  if (g.krange == OZ2_KRANGE_FROM_COL) kt_begin = tn * (TN / BK);
  const int ktiles = kt_end - kt_begin;

  const size_t kp = (size_t)g.k_pad;
  // first byte this wave copies of the tile's first k-tile: tile row r lies in block r / kBlk, TM / 4 rows per wave
  const int8_t* pa = g.a + ((size_t)t * g.m_pad + (size_t)(tm * TM / kBlk) * kBlk) * kp + (size_t)(tm * TM % kBlk) * BK +
                     (size_t)kt_begin * (kBlk * BK) + wv * (TM / 4) * BK;
  const int8_t* pb = g.b + ((size_t)t * g.n_pad + (size_t)(tn * TN / kBlk) * kBlk) * kp + (size_t)(tn * TN % kBlk) * BK +
                     (size_t)kt_begin * (kBlk * BK) + wv * (TN / 4) * BK;
  const unsigned voff = (unsigned)((lane >> 2) * BK) + (((lane & 3) ^ (lane >> 4)) << 4);
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)lds;
  const unsigned lds_a = __builtin_amdgcn_readfirstlane(lds_base + wv * (TM / 4 * BK));
  const unsigned lds_b = __builtin_amdgcn_readfirstlane(lds_base + TM * BK + wv * (TN / 4 * BK));
  auto load = [&](int kt, int st) {
    const size_t off = (size_t)kt * (kBlk * BK);
#pragma unroll
    for (int q = 0; q < kLoadsA; ++q) load_to_lds_16(pa + off + q * 1024, voff, lds_a + st * kStage + q * 1024);
#pragma unroll
    for (int q = 0; q < kLoadsB; ++q) load_to_lds_16(pb + off + q * 1024, voff, lds_b + st * kStage + q * 1024);
  };
  const int swz = (lane >> 2) & 3, half = lane >> 5;
  const int a_off = (wm * (TM / 2) + (lane & 31)) * BK, b_off = TM * BK + (wn * (TN / 2) + (lane & 31)) * BK;
  const int off_s[2] = {((0 + half) ^ swz) << 4, ((2 + half) ^ swz) << 4};

  v16i acc[MI][NI];
#pragma unroll
  for (int x = 0; x < MI; ++x)
#pragma unroll
    for (int y = 0; y < NI; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[x][y][e] = MAXIMA ? 0 : (int)OZ2_ACC_START;
  if (g.fin_stops) fetch_reports(g.fin, lds_base + (NS - 1) * kStage, wv, lane);  // into the stage that the loop fills first
  // (beyond the last k-tile the first one is fetched again: every wait counts on the same number of copies in flight)
#pragma unroll
  for (int p = 0; p < NS - 1; ++p) load(p < ktiles ? p : 0, p);
  if (g.fin_stops) {
    wait_vmcnt<(NS - 2) * kLoads>();
    __syncthreads();
    const int bad = fetched_report_bad(g.fin, lds + (NS - 1) * kStage);
    if (blockIdx.x == 0) write_flags(g.fin, bad);
    if (bad) {
      wait_vmcnt<0>();
      return;
    }
  }
  const Oz2FoldConsts fc = in_vector_registers(g.fold[t]);
  int stage = 0;
  for (int kt = 0; kt < ktiles; ++kt) {
    wait_vmcnt<(NS - 2) * kLoads>();
    __syncthreads();  // k-tile kt is complete, and nobody reads the stage of kt - 1 any more, which is refilled below
    const char* base = lds + stage * kStage;
    v4i fa[2][MI], fb[2][NI];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int x = 0; x < MI; ++x) fa[s][x] = *reinterpret_cast<const v4i*>(base + a_off + x * 32 * BK + off_s[s]);
#pragma unroll
      for (int y = 0; y < NI; ++y) fb[s][y] = *reinterpret_cast<const v4i*>(base + b_off + y * 32 * BK + off_s[s]);
    }
    load(kt + NS - 1 < ktiles ? kt + NS - 1 : 0, stage == 0 ? NS - 1 : stage - 1);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int y = 0; y < NI; ++y)
#pragma unroll
        for (int x = 0; x < MI; ++x)
          acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[s][x], fb[s][y], acc[x][y], 0, 0, 0);
    stage = stage + 1 == NS ? 0 : stage + 1;
  }

  if constexpr (MAXIMA) {
    wait_vmcnt<0>();
    __syncthreads();  // the stages are free
    int* const row_top = reinterpret_cast<int*>(lds);  // [wn][TM], [wm][TN]
    int* const col_top = row_top + 2 * TM;
#pragma unroll
    for (int y = 0; y < NI; ++y) {
      int top = 0;  // (bounds are not negative)
#pragma unroll
      for (int x = 0; x < MI; ++x)
#pragma unroll
        for (int e = 0; e < 16; ++e) top = max(top, acc[x][y][e]);
      top = max(top, __shfl_xor(top, 32, 64));
      if (half == 0) col_top[wm * TN + wn * (TN / 2) + y * 32 + lane] = top;
    }
#pragma unroll
    for (int x = 0; x < MI; ++x) {
      int top[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        top[e] = acc[x][0][e];
#pragma unroll
        for (int y = 1; y < NI; ++y) top[e] = max(top[e], acc[x][y][e]);
      }
      // sixteen rows over 32 lanes: every step halves the rows that a lane keeps
#pragma unroll
      for (int keep = 8, bit = 1; keep >= 1; keep /= 2, bit *= 2)
#pragma unroll
        for (int q = 0; q < keep; ++q) {
          const bool upper = (lane & bit) != 0;
          const int mine = upper ? top[q + keep] : top[q], other = upper ? top[q] : top[q + keep];
          top[q] = max(mine, __shfl_xor(other, bit, 64));
        }
      top[0] = max(top[0], __shfl_xor(top[0], 16, 64));
      const int e = ((lane & 1) << 3) | ((lane & 2) << 1) | ((lane & 4) >> 1) | ((lane & 8) >> 3);
      if ((lane & 16) == 0) row_top[wn * TM + wm * (TM / 2) + x * 32 + 8 * (e >> 2) + 4 * half + (e & 3)] = top[0];
    }
    __syncthreads();
    unsigned long long* const tops = reinterpret_cast<unsigned long long*>(g.c);
    static_assert(TM + TN <= kThreads, "a thread for every row and column");
    const int q = (int)threadIdx.x - TM;
    if (q < 0) {
      const int top = max(row_top[threadIdx.x], row_top[TM + threadIdx.x]);
      if (top > 0) atomicMax(tops + (size_t)tm * TM + threadIdx.x, (unsigned long long)top);
    } else if (q < TN) {
      const int top = max(col_top[q], col_top[TN + q]);
      if (top > 0) atomicMax(tops + (g.triangle != 0 ? 0 : g.m_pad) + (size_t)tn * TN + q, (unsigned long long)top);
    }
    return;
  }

  // Algorithm 1 line 7 (see the large kernel): four consecutive registers are four consecutive rows of a column
  uint8_t* const corner = g.c + ((size_t)t * g.n_pad + (size_t)tn * TN + wn * (TN / 2)) * g.m_pad + (size_t)tm * TM + wm * (TM / 2);
  const unsigned lane_off = (lane & 31u) * (unsigned)g.m_pad + 16u * (lane >> 5);
#pragma unroll
  for (int y = 0; y < NI; ++y) {
    uint8_t* cj = corner + (size_t)(y * 32) * g.m_pad;
    v4i o[MI];
#pragma unroll
    for (int x = 0; x < MI; ++x) {
      unsigned s[16], w[4];
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_udot4((unsigned)acc[x][y][e], fc.kpack, fc.base, false);
#pragma unroll
      for (int a = 0; a < 4; ++a) w[a] = oz2_fold_residues4(s + 4 * a, fc);
      const auto s0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
      o[x] = v4i{(int)s0[0], (int)s0[1], (int)s1[0], (int)s1[1]};
    }
#pragma unroll
    for (int x = 0; x < MI; ++x) *reinterpret_cast<v4i*>(cj + x * 32 + lane_off) = o[x];
  }
  wait_vmcnt<0>();  // the copies fetched beyond the last k-tile must have landed before the LDS is given back
}

template <int MI, int NI, int NS>
constexpr int kTileLds = NS * 64 * (MI + NI) * BK;

template <int MI, int NI, int NS, int WGS, bool WARM, bool MAXIMA = false>
hipError_t set_lds() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_i8_tile_kernel<MI, NI, NS, WGS, WARM, MAXIMA>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds<MI, NI, NS>);
}

// flag: the flag word when the products are not needed once it is set, else null
template <int MI, int NI, int NS, int WGS, bool WARM, bool MAXIMA = false>
hipError_t launch(TileArgs& g, int64_t m, int64_t n, int planes, const unsigned long long* flag, hipStream_t st) {
  constexpr int TM = 64 * MI, TN = 64 * NI;
  g.tiles_m = (int)((m + TM - 1) / TM);
  g.tiles_n = (int)((n + TN - 1) / TN);
  // Symmetric product: only the tiles of the triangle are launched.  (With the other triangle's among them, returning at
  // once, dies and compute units got uneven shares: dsyrk, whole calls, us, 14 moduli, order 900, inner dimension 8192
  // 195 -> 169, 12000 264 -> 227; 16 moduli, order 1837, inner dimension 19821 1084 -> 939.)
  static_assert(TM == TN, "the triangle of a square of tiles");
  g.folded = g.triangle != 0 ? g.tiles_m : 0;
  if (g.folded) fold_triangle(g.folded, &g.tiles_m, &g.tiles_n);
  const int64_t total = (int64_t)g.tiles_m * g.tiles_n * planes;
  if (total > (int64_t)1 << 30) return hipErrorInvalidValue;
  g.total = (int)total;
  g.chunk = (int)((total + 7) / 8);
  g.div_plane = fast_div((unsigned)(g.tiles_m * g.tiles_n));
  g.div_group = fast_div((unsigned)(kGroup * g.tiles_n));
  g.div_last = fast_div((unsigned)(g.tiles_m % kGroup ? g.tiles_m % kGroup : 1));
  g.skip_flag = g.fin.slots ? nullptr : flag;
  // (with reports still to be turned into the flag by this launch, nobody can look at the flag yet)
  const int64_t each = 270 * (g.krange == OZ2_KRANGE_ALL ? g.ktiles : (g.ktiles + 1) / 2) + 600;
  g.fin_stops = 0;
  if (flag && g.fin.slots) {
    const bool wait = total / oz2_gemm_cus() * each >= OZ2_FINISH_FIRST_NS;
    if (g.fin.stops && !wait && g.fin.count <= (unsigned)(TM + TN) * BK / 8u) {
      g.fin_stops = 1;
    } else if (wait || g.fin.stops) {
      if (hipError_t e = oz2_launch_finish_scan(g.fin, st); e != hipSuccess) return e;
      g.fin = {nullptr, 0u, nullptr, 0};
      g.skip_flag = flag;
    }
  }
  hipLaunchKernelGGL((gemm_i8_tile_kernel<MI, NI, NS, WGS, WARM, MAXIMA>), dim3((unsigned)g.chunk * 8), dim3(kThreads),
                     (kTileLds<MI, NI, NS>), st, g);
  return hipGetLastError();
}

#define OZ2_TILE_128 2, 2, 3, 3, true
#define OZ2_TILE_128_MANY 2, 2, 3, 3, false
#define OZ2_TILE_64 1, 1, 4, 4, true
// few workgroups per compute unit, long inner dimensions (launch_tiles)
#define OZ2_TILE_128_ONE 2, 2, 9, 1, true
#define OZ2_TILE_64_ONE 1, 1, 16, 1, true
#define OZ2_TILE_64_TWO 1, 1, 9, 2, true
constexpr int kDeepKtiles = 24;

// tiles of a plane
int64_t tiles_of(int64_t tile, int64_t m, int64_t n, int triangle) {
  const int64_t tm = (m + tile - 1) / tile, tn = (n + tile - 1) / tile;
  return triangle ? tm * (tn + 1) / 2 : tm * tn;
}

}  // namespace

hipError_t oz2_gemm_tiles_setup() {
  hipError_t e = set_lds<OZ2_TILE_128>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_128_MANY>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_64>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_64_ONE>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_64_TWO>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_128_ONE>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_128, true>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_64, true>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_64_ONE, true>();
  if (e == hipSuccess) e = set_lds<OZ2_TILE_64_TWO, true>();
  return e == hipSuccess ? set_lds<OZ2_TILE_128_ONE, true>() : e;
}

static hipError_t launch_tiles(int tile, const Oz2Plan& plan, const Oz2Layout& lay, char* ws, int64_t m, int64_t n, int triangle,
                               int krange, bool check_flag, const Oz2ScanFinish& fin, hipStream_t st) {
  const bool b_is_a = triangle != 0;  // symmetric product
  if (b_is_a && lay.m_pad != lay.n_pad) return hipErrorInvalidValue;
  if (lay.m_pad >= ((int64_t)1 << 27)) return hipErrorInvalidValue;  // the epilogue's lane offsets
  TileArgs g;
  g.a = reinterpret_cast<const int8_t*>(ws + lay.off_a);
  g.b = reinterpret_cast<const int8_t*>(ws + (b_is_a ? lay.off_a : lay.off_b));
  g.c = reinterpret_cast<uint8_t*>(ws + lay.off_c);
  g.m_pad = lay.m_pad;
  g.n_pad = lay.n_pad;
  g.k_pad = lay.k_pad;
  g.ktiles = (int)(lay.k_pad / BK);
  g.triangle = triangle;
  g.krange = krange;
  g.fin = fin;
  const unsigned long long* flag = check_flag ? reinterpret_cast<const unsigned long long*>(ws + lay.off_flags) : nullptr;
  for (int t = 0; t < plan.N; ++t) g.fold[t] = oz2_fold_consts(plan.moduli[t]);
  // Where a compute unit gets one or two workgroups, the copies of a long inner dimension go as far ahead as the LDS allows: with two
  // k-tiles in flight the loop waits for them (whole calls, us: 14 moduli 200 x 200 x 10000 106.3 -> 96.5, 16 moduli 300 x 300 x 2000
  // 38.3 -> 33.3 and x 5000 64.1 -> 53.9, with the smaller tiles in part, dsyrk 500 x 3000 49.5 -> 43.5).
  const int64_t total = tiles_of(tile, m, n, triangle) * plan.N, cus = oz2_gemm_cus();
  const bool deep = g.ktiles >= kDeepKtiles;
  if (tile == 64) {
    if (deep && total <= cus) return launch<OZ2_TILE_64_ONE>(g, m, n, plan.N, flag, st);
    if (deep && total <= 2 * cus) return launch<OZ2_TILE_64_TWO>(g, m, n, plan.N, flag, st);
    return launch<OZ2_TILE_64>(g, m, n, plan.N, flag, st);
  }
  if (deep && total <= cus) return launch<OZ2_TILE_128_ONE>(g, m, n, plan.N, flag, st);
  // With more than eight workgroups per compute unit the constants are fetched where they are needed: the registers of the fetch ahead
  // cost more (whole calls, us, ahead / not: 17 moduli 13728 x 8516 x 167 1655 / 1635, 18 moduli 10028 x 12048 x 192 1821 / 1804; 10
  // moduli 15610 x 64 x 64, five per compute unit, 31.5 / 32.0).
  return total <= 8 * cus ? launch<OZ2_TILE_128>(g, m, n, plan.N, flag, st) : launch<OZ2_TILE_128_MANY>(g, m, n, plan.N, flag, st);
}

// Which kernel's tiles: 64 or 128 (this file) or 256 (oz2_stage2.hip).  64 x 64 when every tile gets a compute unit
// of its own, or half of one where the inner dimension is long.  Otherwise the smaller of two estimates in nanoseconds, whose coefficients are measured times per tile and
// compute unit (a k-tile, and the rest): rounds of the chip with 256 x 256 tiles, which compute the padding, against
// 128 x 128 tiles, of which a compute unit holds three.  Whole calls, 128 against 256 (us): 14 moduli 512^3 24 / 29,
// 700^3 34 / 37, 1024^3 51 / 49, 1024 x 1024 x 2048 87 / 80, 2048^3 212 / 200, 300 x 3000 x 1000 57 / 67, 16 moduli
// 96 x 8192 x 8192 700 / 736, 4096 x 4096 x 1024 469 / 441; 64 against 128: 128^3 16.8 / 17.7, 256^3 18.4 / 19.4, 512^3
// 25.1 / 24.4, 700^3 36 / 34.  The time per k-tile of the small tiles grows from 200 k-tiles on, where their workgroups, which
// nothing keeps on the same k-tiles, read twice the panels from beyond the L2 (whole calls, 128 against 256, us: 8 moduli
// 2048 x 1147 x 9952 376 / 396, 20 moduli 376 x 3560 x 35718 2208 / 2237, 15 moduli 2948 x 270 x 22898 1078 / 1021, 8 moduli
// 1030 x 3420 x 38226 2375 / 2236, 17 moduli 1509 x 700 x 53536 2129 / 1981).  The large tiles' time per k-tile is shorter in a launch of
// three rounds or more, whose workgroups fetch across tiles (17 moduli 1308 x 1848 x 4879 369 / 334, 13 moduli 426 x 5028 x 1066 95.0 / 92.4;
// two rounds, the second nearly empty: 15 moduli 4375 x 165 x 2233 117 / 123, 10 moduli 2656 x 564 x 1231 64 / 71), but not of a triangular
// operand's, which have a workgroup per tile (14 moduli, dtrmm of order 1000 with 2700 columns 86.4 / 93.0).  The rest of their time is
// shorter with the residues of short sums, in launches of five rounds or more, nine with one or two k-tiles (15 moduli 3512 x 2177 x 278 111.2 /
// 100.0, 3122 x 4032 x 257 173 / 162, 12 moduli 3045 x 5324 x 121 164 / 157, 17 moduli 3483 x 1266 x 215 72.4 / 69.5; four rounds, 10 moduli
// 887 x 4989 x 682 77.3 / 81.0, 14 moduli 706 x 5007 x 80 47.7 / 50.7, five 12 moduli 2410 x 2556 x 90 60.0 / 62.4).  Not in a symmetric
// product whose residues' columns are a multiple of 4096 bytes apart, so that the sixteen of a store meet in the same channels (15 moduli,
// order 3996, inner dimension 200, 106.1 / 131.5, 12 moduli 8192 x 161 323 / 367, 12096 x 161 697 / 755; 10240 x 161 496 / 454, general products in
// their other order 13 moduli 12288 x 4096 x 200 552 / 485).
static int tile_size(int64_t m, int64_t n, int64_t k_pad, int num_moduli, int triangle, int krange, int64_t cus) {
  auto rounds = [&](int64_t tile) { return (tiles_of(tile, m, n, triangle) * num_moduli + cus - 1) / cus; };
  if (rounds(64) <= (k_pad / BK >= kDeepKtiles ? 2 : 1)) return 64;
  const int64_t ktiles = krange == OZ2_KRANGE_ALL ? k_pad / BK : (k_pad / BK + 1) / 2;
  const int64_t per_ktile = 270 + (ktiles < 200 ? 0 : ktiles > 445 ? 35 : (ktiles - 200) / 7);
  const int64_t per_large = krange == OZ2_KRANGE_ALL && rounds(256) > 2 ? 660 : 720;
  const bool same_channels = triangle != 0 && (m + 255) / 256 % 16 == 0;
  const bool shorter = krange == OZ2_KRANGE_ALL && rounds(256) > (ktiles > 2 ? 4 : 8) && k_pad <= OZ2_SHORT_SUM && !same_channels;
  const int64_t rest_large = shorter ? 3300 : 4500;
  return rounds(128) * (per_ktile * ktiles + 600) + 3000 < rounds(256) * (per_large * ktiles + rest_large) ? 128 : 256;
}

int oz2_products_tile(const Oz2Plan& plan, const Oz2Layout& lay, int64_t m, int64_t n, int64_t kblock, int residue_u8, int triangle,
                      int krange, int64_t cus) {
  // (the small tiles take UINT8 residues and one block of the inner dimension only)
  const bool fits = residue_u8 && kblock >= lay.k_pad && lay.k_pad <= OZ2_ACC_BLOCK;
  return fits ? tile_size(m, n, lay.k_pad, plan.N, triangle, krange, cus) : 256;
}

hipError_t oz2_launch_products(const Oz2Plan& plan, const Oz2Layout& lay, char* ws, int64_t m, int64_t n, int64_t kblock,
                               int residue_u8, int triangle, int krange, int check_flag, const Oz2ScanFinish& fin,
                               hipStream_t st) {
  const int tile = oz2_products_tile(plan, lay, m, n, kblock, residue_u8, triangle, krange, oz2_gemm_cus());
  if (tile == 256) return oz2_launch_stage2(plan, lay, ws, kblock, residue_u8, triangle, krange, check_flag, fin, st);
  return launch_tiles(tile, plan, lay, ws, m, n, triangle, krange, check_flag != 0, fin, st);
}

// The product of the bound planes, for its row and column maxima.  The smaller tiles wherever they are estimated to take no longer than
// the large ones with their INT32 product, 8 bytes an element, and the launch that reads it
// (15 moduli 3001 x 2777 x 3500 606 -> 580 us a call, where 132 large tiles left half of the chip idle).
int oz2_bound_tile(const Oz2Layout& lay, int64_t m, int64_t n, bool symmetric, int64_t cus) {
  if (lay.m_pad >= ((int64_t)1 << 27) || (symmetric && lay.m_pad != lay.n_pad)) return 256;
  auto rounds = [&](int64_t tile, bool triangle) { return (tiles_of(tile, m, n, triangle) + cus - 1) / cus; };
  const int64_t ktiles = lay.k_pad / BK;
  if (rounds(64, symmetric) <= (ktiles >= kDeepKtiles ? 2 : 1)) return 64;
  const int64_t per_ktile = 270 + (ktiles < 200 ? 0 : ktiles > 445 ? 35 : (ktiles - 200) / 7);
  const int64_t small = rounds(128, symmetric) * (per_ktile * ktiles + 600) + 3000;
  const int64_t large = rounds(256, false) * ((rounds(256, false) > 2 ? 660 : 720) * ktiles + 4500) + lay.m_pad * lay.n_pad / 500 + 5000;
  return small < large ? 128 : 256;
}

hipError_t oz2_launch_bound_maxima(int tile, const Oz2Layout& lay, char* ws, int64_t m, int64_t n, bool symmetric,
                                   const Oz2ScanFinish& fin, hipStream_t st) {
  TileArgs g = {};
  g.a = reinterpret_cast<const int8_t*>(ws + lay.off_a);
  g.b = reinterpret_cast<const int8_t*>(ws + (symmetric ? lay.off_a : lay.off_b));
  g.c = reinterpret_cast<uint8_t*>(ws + lay.off_rownorm);
  g.m_pad = lay.m_pad;
  g.n_pad = lay.n_pad;
  g.k_pad = lay.k_pad;
  g.ktiles = (int)(lay.k_pad / BK);
  g.triangle = symmetric ? 1 : 0;
  g.krange = OZ2_KRANGE_ALL;
  g.fin = fin;
  const int64_t total = tiles_of(tile, m, n, g.triangle), cus = oz2_gemm_cus();
  const bool deep = g.ktiles >= kDeepKtiles;
  if (tile == 64) {
    if (deep && total <= cus) return launch<OZ2_TILE_64_ONE, true>(g, m, n, 1, nullptr, st);
    if (deep && total <= 2 * cus) return launch<OZ2_TILE_64_TWO, true>(g, m, n, 1, nullptr, st);
    return launch<OZ2_TILE_64, true>(g, m, n, 1, nullptr, st);
  }
  if (deep && total <= cus) return launch<OZ2_TILE_128_ONE, true>(g, m, n, 1, nullptr, st);
  return launch<OZ2_TILE_128, true>(g, m, n, 1, nullptr, st);
}

void oz2_host_product_residues_impl(int p, int64_t count, const int32_t* products, uint8_t* out) {
  const Oz2FoldConsts c = oz2_fold_consts(p);
  for (int64_t i = 0; i < count; ++i) out[i] = oz2_host_fold_residue(products[i], c);
}
void oz2_host_short_product_residues_impl(int p, int64_t count, const int32_t* products, uint8_t* out) {
  const Oz2FoldConsts c = oz2_fold_consts(p);
  for (int64_t i = 0; i < count; ++i) out[i] = oz2_host_short_residue(products[i], c);
}
