// Stage 1b and stage 2 in one kernel for thin products (Algorithm 1 lines 2-7): a large operand against at most 128 vectors
// of the other one.
//
// The residue planes of the large operand are N bytes per element that the conversion writes and the products read once:
// at 8192 x 96 x 8192 with 16 moduli the 1.1 GB of planes cost two thirds of the call.  Here a workgroup takes 64 vectors
// of the large operand and a group of up to eight moduli, converts a k-tile of 64 inner positions at a time in registers,
// passes the residues through LDS (64 rows x 64 bytes per modulus) and multiplies them with the planes
// of the thin operand, which come straight from the L2 in the layout an MFMA operand has: wave w works for modulus w of the
// group and nobody else needs those bytes.  The large operand is read once per group (the groups of the same 64 vectors
// run on the same die at the same time and find it in the L2); its planes do not exist.
// Bound by the conversion's vector instructions and by waits: 336 instructions of 4.5 cycles per wave and k-tile, two waves per
// SIMD, are 3000 of its 4400 cycles (16 moduli 8192 x 96 x 8192).  The loop has no branch that loads, and its loads stay where
// they are written: left to itself the compiler moves them down to their use, where their latency shows (475 -> 406 us a call
// there).  Two k-tiles share a barrier, the large operand is fetched two k-tiles ahead into the registers just split, and the
// products stand between the steps of the conversion, which the matrix cores work beside (a k-tile per barrier, products ahead of the
// conversion / this, us: 16 moduli 8192 x 96 x 8192 389 / 366, 96 x 8192 x 8192 419 / 399, 8192 x 32 x 8192 348 / 327, 18 moduli
// 8192 x 96 x 8192 575 / 520, 14 moduli 64 x 15484 x 9445 905 / 818).  The order of the two fetches matters: with the large operand's
// behind the thin one's 96 x 8192 x 8192 takes 450.
//
// 512 threads, eight waves, two per SIMD: 32 NI accumulators per lane (NI = 32-vector tiles of the thin operand), ordinary
// registers (build.py builds this file with -amdgpu-mfma-vgpr-form).
#include <type_traits>

#include "oz2_gemm.h"
#include "oz2_math.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kThreads = 512;
constexpr int kRows = 64;               // vectors of the large operand per workgroup
constexpr int kGroup = kThreads / 64;   // moduli per group: one per wave
constexpr int BK = OZ2_TILE_K;
constexpr int kBlk = OZ2_TILE_M;        // plane layout: blocks of 256 rows x 64 bytes
constexpr int kTileBytes = kRows * BK;  // one modulus in LDS
constexpr int kMaxThin = 128;
template <int KIND, bool PAIRED>
constexpr bool kArray = !PAIRED && KIND == 0;
template <int KIND, bool PAIRED>
constexpr int kThinLds = kArray<KIND, PAIRED> ? 0 : (PAIRED ? 4 : 2) * kGroup * kTileBytes;  // of the launch's own size
constexpr int kMfmaSteps = 8;           // steps of a k-tile's conversion that carry its products

struct ThinArgs {
  const double* X;        // large operand: element (v, l) at X[v + l ld] (strided) or X[l + v ld]
  int64_t ld, nvec, k;
  const int* shifts;
  int strided;
  const int8_t* thin;     // planes of the thin operand
  int64_t thin_pad, k_pad;
  uint8_t* c;
  int64_t m_pad, n_pad;
  int groups, per_group;  // groups of moduli
  int total, chunk;       // workgroups, and workgroups per die
  FastDiv div_groups;
  const unsigned long long* skip_flag;
  Oz2ConvConsts conv;
  Oz2FoldConsts fold[OZ2_MAX_N];
};

template <int KIND, int NI, bool BIG_A, bool PAIRED>
__global__ void __launch_bounds__(kThreads) thin_products_kernel(const ThinArgs g) {
  constexpr bool TWO_LEVEL = KIND == 1;
  // The k-tiles in LDS: of the launch's own size, or two in an array, for which the compiler makes another schedule: the better one for
  // elements split one level deep (16 moduli 128 x 5824 x 14528 785 -> 766 us a call, 18 moduli 128 x 8195 x 9097 968 -> 929), not for
  // two (22 moduli 8192 x 128 x 8192 788 -> 826).
  constexpr bool ARRAY = kArray<KIND, PAIRED>;
  extern __shared__ __attribute__((aligned(1024))) char thin_lds[];
  auto own = reinterpret_cast<char(*)[kGroup][kTileBytes]>(thin_lds);
  __shared__ __attribute__((aligned(1024))) char two[ARRAY ? 2 : 1][ARRAY ? kGroup : 1][ARRAY ? kTileBytes : 16];
  if (g.skip_flag != nullptr && *g.skip_flag != 0ull) return;
  const int item = (int)(blockIdx.x & 7) * g.chunk + (int)(blockIdx.x >> 3);  // workgroup i of a launch runs on die i % 8
  if (item >= g.total) return;
  const int rg = item / g.div_groups, group = item - rg * g.groups;
  const int64_t r0 = (int64_t)rg * kRows;
  const int t0 = group * g.per_group;
  const int count = min(g.per_group, g.conv.N - t0);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // ---- conversion: this thread's vector and its eight inner positions of a k-tile
  const int row = g.strided ? lane : 8 * wv + (lane >> 3);
  const int pos = g.strided ? 8 * wv : 8 * (lane & 7);
  // (a workgroup's last rows may lie beyond the operand: they repeat its last vector, and nobody reads their results)
  const int64_t v = r0 + row < g.nvec ? r0 + row : g.nvec - 1;
  const int shift = g.shifts[v];
  const double* const src = g.strided ? g.X + v + (int64_t)pos * g.ld : g.X + v * g.ld + pos;
  const int64_t step = g.strided ? g.ld : 1;
  const int ktiles = (int)(g.k_pad / BK);
  auto fetch = [&](int kt, auto whole, double (&d)[8]) {
    const double* p = src + (int64_t)kt * BK * step;
    if constexpr (decltype(whole)::value) {
#pragma unroll
      for (int u = 0; u < 8; ++u) d[u] = p[u * step];
    } else {  // the last k-tile, or beyond it: the last element where there is nothing to read, then zero instead
      const int last = (int)(g.k - ((int64_t)kt * BK + pos)) - 1;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double x = p[min(u, last) * step];
        d[u] = u <= last ? x : 0.0;
      }
    }
  };
  // 16-byte chunks of a row are swizzled as in the GEMM's stages (fragments of 16 rows fall on 16 bank groups)
  const int put = row * BK + ((((pos >> 4) ^ (row >> 2)) & 3) << 4) + (pos & 8);
  Oz2ConvMod mods[kGroup];  // in scalar registers throughout (loaded per k-tile, every modulus waited for its constants)
#pragma unroll
  for (int tt = 0; tt < kGroup; ++tt) mods[tt] = g.conv.mod[tt < count ? t0 + tt : t0];
  // one k-tile in twelve steps: four that split two elements each, one per modulus; after(step) is called between them
  auto convert = [&](const double (&d)[8], int buf, auto&& after) {
    Oz2SplitPair<TWO_LEVEL> xs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      xs[u] = oz2_split_pair<TWO_LEVEL>(d[2 * u], d[2 * u + 1], shift);
      after(u);
    }
#pragma unroll
    for (int tt = 0; tt < kGroup; ++tt) {
      if (tt < count) {
        v2u w;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          w[h] = oz2_pack_pairs(oz2_residue_pair<TWO_LEVEL>(xs[2 * h], mods[tt]),
                                oz2_residue_pair<TWO_LEVEL>(xs[2 * h + 1], mods[tt]));
        if constexpr (ARRAY)
          *reinterpret_cast<v2u*>(&two[buf][tt][put]) = w;
        else
          *reinterpret_cast<v2u*>(&own[buf][tt][put]) = w;
      }
      after(4 + tt);
    }
  };

  // ---- products: wave w for modulus t0 + w
  const bool works = wv < count;
  const int t = works ? t0 + wv : t0;
  const int half = lane >> 5, swz = (lane >> 2) & 3;
  const int8_t* const thin = g.thin + (size_t)t * g.thin_pad * g.k_pad + (lane & 31) * BK + half * 16;
  v4i ft[2][NI];
  auto fetch_thin = [&](int kt) {
    const int8_t* p = thin + (size_t)kt * (kBlk * BK);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int y = 0; y < NI; ++y) ft[s][y] = *reinterpret_cast<const v4i*>(p + y * 32 * BK + s * 32);
  };
  v16i acc[2][NI];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < NI; ++y)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[x][y][e] = (int)OZ2_ACC_START;

  auto fragments = [&](int slot, v4i (&fb)[2][2]) {
    const char* base;
    if constexpr (ARRAY)
      base = two[slot][works ? wv : 0] + (lane & 31) * BK;
    else
      base = own[slot][works ? wv : 0] + (lane & 31) * BK;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x)
        fb[s][x] = *reinterpret_cast<const v4i*>(base + x * 32 * BK + (((2 * s + half) ^ swz) << 4));
  };
  auto multiply = [&](const v4i (&fb)[2][2], int from, int to) {
#pragma unroll
    for (int q = from; q < to; ++q) {
      const int s = q / (2 * NI), y = q / 2 % NI, x = q % 2;
      acc[x][y] = BIG_A ? __builtin_amdgcn_mfma_i32_32x32x32_i8(fb[s][x], ft[s][y], acc[x][y], 0, 0, 0)
                        : __builtin_amdgcn_mfma_i32_32x32x32_i8(ft[s][y], fb[s][x], acc[x][y], 0, 0, 0);
    }
  };
  const std::true_type whole;
  const std::false_type part;
  double d0[8], d1[8];
  fetch(0, whole, d0);  // (the inner dimension is above 1024)
  fetch(1, whole, d1);
  fetch_thin(0);
  convert(d0, 0, [](int) {});
  int kt = 0;  // two k-tiles in a round; what lies beyond the last one is zero
  if constexpr (PAIRED) {
    // k-tiles kt and kt + 1 are multiplied while kt + 2 and kt + 3 are converted and kt + 4 and kt + 5 are on their way from
    // memory, one barrier for the two.  No branches: where paths that load join, or a loop-carried value is copied, the loads
    // in flight are waited for.
    auto iteration = [&](int kt, auto whole, double (&d)[8]) {
      v4i fb[2][2];
      fragments(kt & 3, fb);
      convert(d, (kt + 2) & 3, [&](int step) {
        if (step < kMfmaSteps) {
          __builtin_amdgcn_sched_barrier(0);
          multiply(fb, 4 * NI * step / kMfmaSteps, 4 * NI * (step + 1) / kMfmaSteps);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (step == 3) {  // the elements are split: their registers take the next ones
          fetch(kt + 4, whole, d);
          asm volatile("" ::: "memory");  // (the compiler would move the loads down to where their results are needed)
        }
        if (step == kMfmaSteps - 1) {
          fetch_thin(kt + 1 < ktiles ? kt + 1 : ktiles - 1);
          asm volatile("" ::: "memory");
        }
      });
    };
    fetch(2, whole, d0);
    convert(d1, 1, [](int) {});
    fetch(3, whole, d1);
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): what is pending here would be waited for in every round of the loop
    for (; (int64_t)(kt + 6) * BK <= g.k; kt += 2) {
      iteration(kt, whole, d0);
      iteration(kt + 1, whole, d1);
      __syncthreads();  // the next two k-tiles are complete, and nobody reads these two any more
    }
    for (; kt < ktiles; kt += 2) {
      iteration(kt, part, d0);
      iteration(kt + 1, part, d1);
      __syncthreads();
    }
  } else {
    // k-tile kt is multiplied, then kt + 1 is converted, while kt + 2 is on its way from memory: 16 registers less
    auto iteration = [&](int kt, int slot, auto whole, const double (&now)[8], double (&later)[8]) {
      fetch(kt + 2, whole, later);
      asm volatile("" ::: "memory");
      v4i fb[2][2];
      fragments(slot, fb);
      multiply(fb, 0, 4 * NI);
      fetch_thin(kt + 1 < ktiles ? kt + 1 : ktiles - 1);
      asm volatile("" ::: "memory");
      convert(now, slot ^ 1, [](int) {});
      __syncthreads();  // the next k-tile is complete, and nobody reads this one's slot any more
    };
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0f70);
    for (; (int64_t)(kt + 4) * BK <= g.k; kt += 2) {
      iteration(kt, 0, whole, d1, d0);
      iteration(kt + 1, 1, whole, d0, d1);
    }
    for (; kt < ktiles; kt += 2) {
      iteration(kt, 0, part, d1, d0);
      iteration(kt + 1, 1, part, d0, d1);
    }
  }
  if (!works) return;

  // ---- residues (Algorithm 1 line 7, see the GEMM's epilogue): a lane holds column lane % 32 of a 32 x 32 tile
  const Oz2FoldConsts fc = in_vector_registers(g.fold[t]);
  uint8_t* const plane = g.c + (size_t)t * g.n_pad * g.m_pad + (size_t)(lane & 31) * g.m_pad + 16 * half;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < NI; ++y) {
      unsigned s[16], w[4];
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_udot4((unsigned)acc[x][y][e], fc.kpack, fc.base, false);
#pragma unroll
      for (int a = 0; a < 4; ++a) w[a] = oz2_fold_residues4(s + 4 * a, fc);
      const auto s0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
      const int64_t i = BIG_A ? r0 + x * 32 : y * 32, j = BIG_A ? y * 32 : r0 + x * 32;
      *reinterpret_cast<v4i*>(plane + j * g.m_pad + i) = v4i{(int)s0[0], (int)s0[1], (int)s1[0], (int)s1[1]};
    }
}

// Which form: pairs of k-tiles where their registers and 128 KiB of LDS cost nothing, one at a time for four tiles of the thin
// operand (the pairs would keep 84 to 270 bytes per lane in scratch memory: 8192 x 128 x 8192 with 16 moduli 426 -> 527 us) and
// for one tile with the one-level split when there are workgroups for two on a compute unit, which fit then (16384 x 32 x 4096
// 315 us, in pairs 331).
template <int KIND, int NI>
constexpr bool kPairs = NI < 4;
template <int KIND, int NI>
constexpr bool kSingles = NI == 4 || (NI == 1 && KIND == 0);

template <int KIND, int NI, bool PAIRED>
hipError_t set_thin_lds() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(thin_products_kernel<KIND, NI, true, PAIRED>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kThinLds<KIND, PAIRED>);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(thin_products_kernel<KIND, NI, false, PAIRED>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kThinLds<KIND, PAIRED>);
}
template <int KIND, int NI>
hipError_t set_thin() {
  hipError_t e = hipSuccess;
  if constexpr (kPairs<KIND, NI>) e = set_thin_lds<KIND, NI, true>();
  if constexpr (kSingles<KIND, NI> && !kArray<KIND, false>) e = e == hipSuccess ? set_thin_lds<KIND, NI, false>() : e;
  return e;
}
template <int KIND>
hipError_t set_thin_kind() {
  hipError_t e = set_thin<KIND, 1>();
  if (e == hipSuccess) e = set_thin<KIND, 2>();
  if (e == hipSuccess) e = set_thin<KIND, 3>();
  return e == hipSuccess ? set_thin<KIND, 4>() : e;
}

template <int KIND, int NI, bool BIG_A>
void launch_thin(const ThinArgs& g, hipStream_t st) {
  const dim3 grid((unsigned)g.chunk * 8), thr(kThreads);
  const bool two_fit = g.total > oz2_gemm_cus();
  if constexpr (kPairs<KIND, NI> && kSingles<KIND, NI>) {
    if (two_fit) {
      hipLaunchKernelGGL((thin_products_kernel<KIND, NI, BIG_A, false>), grid, thr, (kThinLds<KIND, false>), st, g);
      return;
    }
  }
  hipLaunchKernelGGL((thin_products_kernel<KIND, NI, BIG_A, kPairs<KIND, NI>>), grid, thr, (kThinLds<KIND, kPairs<KIND, NI>>), st, g);
}

}  // namespace

// Once per process, before any launch: the dynamic LDS limits.
hipError_t oz2_thin_setup() {
  const hipError_t e = set_thin_kind<0>();
  return e == hipSuccess ? set_thin_kind<1>() : e;
}

// The smaller of two estimates in nanoseconds, measured times per k-tile of a workgroup (one per compute unit) and per
// byte that conversion and products move between them otherwise (8 read, N written, N read per element of the large
// operand, 4.3 TB/s).  Whole calls, with planes against without (us): 16 moduli 8192 x 96 x 8192 680 / 366, 96 x 8192 x 8192
// 698 / 399, 8192 x 32 x 8192 671 / 327, 16384 x 64 x 2048 374 / 195; 14 moduli 64 x 15484 x 9445 1391 / 818; 18 moduli
// 8192 x 96 x 8192 739 / 520; 22 moduli 8192 x 96 x 8192 906 / 702.
int oz2_thin_applies(int64_t m, int64_t n, const Oz2Plan& plan, const Oz2Layout& lay, int64_t kblock, int64_t cus) {
  const int64_t thin = m < n ? m : n, large = m < n ? n : m;
  // (up to 1024 the one-pass conversion reads the operand once, which is the better half of this; above, where it does so too up to 9920,
  // these kernels are still ahead where this rule takes them, whole calls, one pass / here, us: 16 moduli 8192 x 96 x 2000 189 / 114,
  // 96 x 8192 x 2000 157 / 117, 12 moduli 16000 x 90 x 1500 210 / 145)
  if (thin > kMaxThin || lay.k_pad <= 1024 || lay.k_pad > OZ2_ACC_BLOCK || kblock < lay.k_pad) return 0;
  const int64_t groups = (plan.N + kGroup - 1) / kGroup;
  const int64_t rounds = ((large + kRows - 1) / kRows * groups + cus - 1) / cus;
  const int64_t here = rounds * (lay.k_pad / BK) * 2400, planes = large * lay.k_pad / 10 * (8 + 2 * plan.N) / 430;
  return here < planes - planes / 10 ? (m < n ? 2 : 1) : 0;
}

hipError_t oz2_launch_thin_products(int which, int strided, const double* X, int64_t ld, int64_t nvec, int64_t nthin, int64_t k,
                                    int two_level, const Oz2Plan& plan, const Oz2Layout& lay, char* ws, int check_flag,
                                    hipStream_t st) {
  if (nthin > kMaxThin) return hipErrorInvalidValue;
  const bool big_a = which == 1;
  ThinArgs g;
  g.X = X;
  g.ld = ld;
  g.nvec = nvec;
  g.k = k;
  g.shifts = reinterpret_cast<const int*>(ws + (big_a ? lay.off_sa : lay.off_sb));
  g.strided = strided;
  g.thin = reinterpret_cast<const int8_t*>(ws + (big_a ? lay.off_b : lay.off_a));
  g.thin_pad = big_a ? lay.n_pad : lay.m_pad;
  g.k_pad = lay.k_pad;
  g.c = reinterpret_cast<uint8_t*>(ws + lay.off_c);
  g.m_pad = lay.m_pad;
  g.n_pad = lay.n_pad;
  g.groups = (plan.N + kGroup - 1) / kGroup;
  g.per_group = (plan.N + g.groups - 1) / g.groups;
  const int64_t total = (nvec + kRows - 1) / kRows * g.groups;
  if (total > (int64_t)1 << 30) return hipErrorInvalidValue;
  g.total = (int)total;
  g.chunk = (int)((total + 7) / 8);
  g.div_groups = fast_div((unsigned)g.groups);
  g.skip_flag = check_flag ? reinterpret_cast<const unsigned long long*>(ws + lay.off_flags) : nullptr;
  g.conv = plan.conv;
  for (int t = 0; t < plan.N; ++t) g.fold[t] = oz2_fold_consts(plan.moduli[t]);
  const int ni = (int)((nthin + 31) / 32);
#define OZ2_THIN(KIND, NI) (big_a ? launch_thin<KIND, NI, true>(g, st) : launch_thin<KIND, NI, false>(g, st))
#define OZ2_THIN_NI(KIND)                                                                    \
  do {                                                                                       \
    if (ni == 1)                                                                             \
      OZ2_THIN(KIND, 1);                                                                     \
    else if (ni == 2)                                                                        \
      OZ2_THIN(KIND, 2);                                                                     \
    else if (ni == 3)                                                                        \
      OZ2_THIN(KIND, 3);                                                                     \
    else                                                                                     \
      OZ2_THIN(KIND, 4);                                                                     \
  } while (0)
  if (two_level)
    OZ2_THIN_NI(1);
  else
    OZ2_THIN_NI(0);
#undef OZ2_THIN_NI
#undef OZ2_THIN
  return hipGetLastError();
}
