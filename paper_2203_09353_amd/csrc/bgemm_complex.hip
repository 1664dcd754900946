// Complex batched GEMM (the paper's matrices are complex, Section II, Eq. 1):
// C_i <- alpha op(A_i) op(B_i) + beta C_i with interleaved binary64 (real,
// imaginary) elements, op = N, T or C (conjugate transpose).
//
// Four real products per complex one, on the FP64 matrix cores:
//     Re C += Re a Re b - Im a Im b,   Im C += Re a Im b + Im a Re b
// with a = op(A)(r, p), b = op(B)(p, c).  An element is one 16-byte unit from
// global memory to the fragment registers: operand tiles go straight to LDS
// as they are (no expansion into real and imaginary planes, no staging
// registers) and one 16-byte LDS read feeds both parts.  Signs, conjugation
// included, are flipped on the sixteen-row fragments just before use.
//
// One v_mfma_f64_4x4x4_4b_f64 takes a 16-row slab of op(A) (lane 16 s + r
// holds row r at k s) and four columns of op(B) replicated over its four
// blocks (lane 16 s + 4 b + j holds column j), and yields a 16 x 4 block of C's
// real or imaginary parts (lane 16 i + 4 b + j holds row 4 b + i, column j).
// The two parts go to two accumulators, so both parts of a C element sit in
// one lane for the complex epilogue, and a lane group's sixteen rows are 256
// contiguous bytes of a C column.
//
// Tile: 64 x 64 complex C per workgroup (64 x 32 or 64 x 16 for fewer columns),
// a wave per 16 columns, eight complex k per step, a ring of three LDS stages
// filled by direct global-to-LDS loads two steps ahead, three workgroups per CU
// (four or five of the narrow ones).  What bounds it: the matrix cores
// (a 256 x 256 x 128 product moves 1.57 MB for 67 MFLOP).
// Measured: 10,000 x Psi Psi^H of 256 x 128 12.8 -> 10.5 ms (52.5 -> 64 TFLOP/s),
// 64 of 2048 x 1024 38.6 -> 32.2 ms (68 TFLOP/s), 3,000 x 200 x 90 x 300 conjugated
// 4.63 -> 3.48, 10,000 x 16 x 16 x 100 0.58 -> 0.15, against register-staged planes
// of an embedded real operand.  128 x 64 tiles of eight waves ran 11.9 ms (two
// waves per SIMD), 32 x 16 waves 10.85, two workgroups per CU 11.0.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bgemm_internal.h"

namespace bg {
namespace cplx {

#define AS_GLOBAL __attribute__((address_space(1)))
#define AS_LDS __attribute__((address_space(3)))
typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));  // at any 8-byte boundary
typedef const AS_GLOBAL double* gcptr;
typedef AS_LDS d2* uptr;             // a 16-byte unit in LDS: one complex element
typedef const AS_LDS d2* ucptr;

constexpr int BM = 64, BK = 8, NS = 3;
constexpr int WM = 64, WN = 16, FP = WM / 16, GQ = WN / 4;
static_assert(BM == WM, "one wave per 16 columns");

// s_waitcnt immediate: vector-memory count vm, LDS/scalar count lgkm, export
// count unconstrained (gfx9 encoding)
constexpr int waitcnt_imm(int vm, int lgkm) {
  return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm & 15) << 8);
}

__device__ __forceinline__ double flip(double x) {
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, x) ^ (1ull << 63));
}

// An operand tile in LDS: EXT values of its product dimension x BK of k, units
// in the operand's own order.  MN-contiguous: row k of EXT units (a fragment
// read's sixteen rows are 256 contiguous bytes).  K-contiguous: rows of BK = 8
// units, XOR-swizzled by (row / 2) mod 8 so that sixteen rows read at one k
// fall in sixteen distinct 16-byte bank groups.
template <int EXT, bool KC>
struct Tile {
  static constexpr int UNITS = EXT * BK;
  __device__ __forceinline__ static int pos(int mn, int k) {
    return KC ? mn * BK + (k ^ ((mn >> 1) & 7)) : k * EXT + mn;
  }
  // the element that unit u holds
  __device__ __forceinline__ static void at(int u, int& mn, int& k) {
    if (KC) {
      mn = u / BK;
      k = (u % BK) ^ ((mn >> 1) & 7);
    } else {
      mn = u % EXT;
      k = u / EXT;
    }
  }
};

// Three waves per SIMD (three 64-wide workgroups per CU, as many as the LDS
// holds) need at most 170 registers, two (the narrow tiles) 256, which the
// compiler reaches without a spill (the build checks: a spill would enter the
// counted waits).
template <int TA, int TB, int BN>
__global__ __launch_bounds__(BN * 4, BN == 64 ? 3 : 2) void k_uniform_z(
    int M, int N, int K, double ar, double ai, const double* const* __restrict__ Ap, int64_t lda,
    const double* const* __restrict__ Bp, int64_t ldb, double br, double bi,
    double* const* __restrict__ Cp, int64_t ldc, int tiles_m, int tiles_per_inst,
    int64_t total_tiles, int64_t per_xcd) {
  // the epilogue's complex products round as written (no fused multiply-add)
#pragma clang fp contract(off)
  constexpr int NT = BN * 4, NW = NT / 64;
  constexpr int PA = BM * BK / NT, PB = BN * BK / NT;   // units per thread and step
  constexpr int DPT = PA + PB;                          // its direct loads per step
  constexpr int STAGE = (BM + BN) * BK;                 // units
  using TAt = Tile<BM, TA != 0>;
  using TBt = Tile<BN, TB == 0>;
  __shared__ __align__(16) double lds_raw[2 * NS * STAGE];
  const uptr lds = (uptr)lds_raw;
  const int64_t bid = blockIdx.x;
  const int64_t id = (bid % 8) * per_xcd + bid / 8;   // contiguous tiles per XCD
  if (id >= total_tiles) return;
  const int64_t inst = id / tiles_per_inst;
  const int tt = (int)(id - inst * tiles_per_inst);
  const int m0 = (tt % tiles_m) * BM, n0 = (tt / tiles_m) * BN;
  const gcptr A = (gcptr)Ap[inst];
  const gcptr B = (gcptr)Bp[inst];
  AS_GLOBAL double* C = (AS_GLOBAL double*)Cp[inst];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn0 = wave * WN;
  const int ls = lane >> 4, lr = lane & 15, lj = lane & 3;

  // This thread's units of a stage, as element offsets from (k = 0) and the
  // step's advance.  Units outside the matrix re-read the tile's first row or
  // column: in bounds, every wave issues the same number of direct loads (the
  // stage waits count them), and their products only reach C elements outside
  // C.
  int64_t oa[PA], ob[PB];
  int ka[PA], kb[PB];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    int mn;
    TAt::at((i * NW + wave) * 64 + lane, mn, ka[i]);
    const int64_t r = m0 + mn < M ? m0 + mn : m0;
    oa[i] = TA == 0 ? r + ka[i] * lda : ka[i] + r * lda;
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    int mn;
    TBt::at((i * NW + wave) * 64 + lane, mn, kb[i]);
    const int64_t c = n0 + mn < N ? n0 + mn : n0;
    ob[i] = TB == 0 ? kb[i] + c * ldb : c + kb[i] * ldb;
  }
  const int64_t sa = TA == 0 ? BK * lda : BK, sb = TB == 0 ? BK : BK * ldb;
  const int nk = (K + BK - 1) / BK;
  const bool tail = K % BK != 0;

  auto issue = [&](int kt, int st) {
    const uptr la = lds + st * STAGE, lb = la + TAt::UNITS;
    if (kt == nk - 1 && tail) {
      // partial in k: through registers, zero beyond K.  Every load is
      // unconditional (k clamped), and the explicit wait also covers the
      // direct loads issued before it, whatever this wave's lanes hold.
      const int k0 = kt * BK;
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        const int over = k0 + ka[i] >= K ? k0 + ka[i] - (K - 1) : 0;
        const d2 x = *(const AS_GLOBAL d2u*)(A + 2 * (oa[i] + kt * sa - over * (TA == 0 ? lda : 1)));
        la[(i * NW + wave) * 64 + lane] = over ? d2{0.0, 0.0} : x;
      }
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        const int over = k0 + kb[i] >= K ? k0 + kb[i] - (K - 1) : 0;
        const d2 x = *(const AS_GLOBAL d2u*)(B + 2 * (ob[i] + kt * sb - over * (TB == 0 ? 1 : ldb)));
        lb[(i * NW + wave) * 64 + lane] = over ? d2{0.0, 0.0} : x;
      }
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    } else {
#pragma unroll
      for (int i = 0; i < PA; ++i)
        __builtin_amdgcn_global_load_lds((const AS_GLOBAL void*)(A + 2 * (oa[i] + kt * sa)),
                                         (AS_LDS void*)(la + (i * NW + wave) * 64), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < PB; ++i)
        __builtin_amdgcn_global_load_lds((const AS_GLOBAL void*)(B + 2 * (ob[i] + kt * sb)),
                                         (AS_LDS void*)(lb + (i * NW + wave) * 64), 16, 0, 0);
    }
  };

  // acc[t][g]: slab t (16 rows), column group g (4), real and imaginary parts
  double cr[FP][GQ], ci[FP][GQ];
#pragma unroll
  for (int t = 0; t < FP; ++t)
#pragma unroll
    for (int g = 0; g < GQ; ++g) cr[t][g] = ci[t][g] = 0.0;

#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < nk) issue(st, st);

  // Step kt lives in stage kt mod NS.  Its loads are complete once at most the
  // next step's DPT loads remain (they return in order); the barrier then
  // publishes every wave's part, and only after it is the stage read one step
  // earlier refilled.  NPA of the wave's slabs take part (fewer on edge tiles,
  // none for a wave outside C); every wave issues the same loads and barriers.
  auto step = [&](int kt, auto stage_c, auto npa_c) {
    constexpr int st = decltype(stage_c)::value;
    constexpr int NPA = decltype(npa_c)::value;
    asm volatile("" ::: "memory");
    if (kt + 1 < nk) __builtin_amdgcn_s_waitcnt(waitcnt_imm(DPT, 0));
    else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_setprio(1);
    auto refill = [&]() {
      asm volatile("" ::: "memory");
      if (kt + NS - 1 < nk) issue(kt + NS - 1, (st + NS - 1) % NS);
      asm volatile("" ::: "memory");
    };
    if constexpr (NPA == 0) refill();
    const ucptr la = lds + st * STAGE, lb = la + TAt::UNITS;
    if constexpr (NPA > 0) {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        d2 p[NPA], q[GQ];
#pragma unroll
        for (int t = 0; t < NPA; ++t) p[t] = la[TAt::pos(16 * t + lr, kk + ls)];
#pragma unroll
        for (int g = 0; g < GQ; ++g) q[g] = lb[TBt::pos(wn0 + 4 * g + lj, kk + ls)];
        if (kk == 4) refill();
#pragma unroll
        for (int t = 0; t < NPA; ++t) {
          // signs: Re takes -Im a Im b, or + when exactly one is conjugated;
          // Im takes Re a Im b negated for conj b, Im a Re b negated for conj a
          const double pr = p[t].x, pi = p[t].y;
          const double pir = (TA == 2) == (TB == 2) ? flip(pi) : pi;
          const double pri = TB == 2 ? flip(pr) : pr;
          const double pii = TA == 2 ? flip(pi) : pi;
#pragma unroll
          for (int g = 0; g < GQ; ++g) {
            cr[t][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(pr, q[g].x, cr[t][g], 0, 0, 0);
            ci[t][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(pri, q[g].y, ci[t][g], 0, 0, 0);
          }
#pragma unroll
          for (int g = 0; g < GQ; ++g) {
            cr[t][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(pir, q[g].y, cr[t][g], 0, 0, 0);
            ci[t][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(pii, q[g].x, ci[t][g], 0, 0, 0);
          }
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
  };
  auto kloop = [&](auto npa_c) {
    for (int kt = 0; kt < nk; kt += NS) {
      step(kt, std::integral_constant<int, 0>{}, npa_c);
      if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>{}, npa_c);
      if (kt + 2 < nk) step(kt + 2, std::integral_constant<int, 2>{}, npa_c);
    }
  };
  const int slabs = n0 + wn0 < N ? (M - m0 + 15) / 16 : 0;
  using std::integral_constant;
  static_assert(FP == 4, "slab counts below");
  if (slabs >= 4) kloop(integral_constant<int, 4>{});
  else if (slabs == 3) kloop(integral_constant<int, 3>{});
  else if (slabs == 2) kloop(integral_constant<int, 2>{});
  else if (slabs == 1) kloop(integral_constant<int, 1>{});
  else kloop(integral_constant<int, 0>{});

  // Epilogue: lane 16 i + 4 b + j holds row 16 t + 4 b + i, column
  // wn0 + 4 g + j of slab t, group g.
  const bool read_c = !(br == 0.0 && bi == 0.0);
  const int row0 = m0 + 4 * ((lane >> 2) & 3) + (lane >> 4);
  // Every value of C is asked for before the first is used: 8,003 x 107 x 64 x 14
  // with beta 1 took 567 us a column group at a time, 427 so.
  d2 cv[GQ][FP];
  if (read_c) {
#pragma unroll
    for (int g = 0; g < GQ; ++g)
#pragma unroll
      for (int t = 0; t < FP; ++t) {
        const int c = n0 + wn0 + 4 * g + lj;
        if (row0 + 16 * t < M && c < N)
          cv[g][t] = *(const AS_GLOBAL d2u*)(C + 2 * (row0 + 16 * t + (int64_t)c * ldc));
      }
  }
#pragma unroll
  for (int g = 0; g < GQ; ++g)
#pragma unroll
    for (int t = 0; t < FP; ++t) {
      const int c = n0 + wn0 + 4 * g + lj;
      if (row0 + 16 * t >= M || c >= N) continue;
      d2 x{ar * cr[t][g] - ai * ci[t][g], ar * ci[t][g] + ai * cr[t][g]};
      if (read_c) {
        x.x = x.x + (br * cv[g][t].x - bi * cv[g][t].y);
        x.y = x.y + (br * cv[g][t].y + bi * cv[g][t].x);
      }
      *(AS_GLOBAL d2u*)(C + 2 * (row0 + 16 * t + (int64_t)c * ldc)) = x;
    }
}

// C <- beta C (complex), exactly zero when beta == 0 (C not read).
__global__ __launch_bounds__(256) void k_zscale(double br, double bi, double* const* __restrict__ Cp,
                                                int64_t ldc, int m, int n, int64_t total_cols) {
#pragma clang fp contract(off)
  for (int64_t col = blockIdx.x; col < total_cols; col += gridDim.x) {
    const int64_t inst = col / n;
    const int c = (int)(col - inst * n);
    double* base = Cp[inst] + 2 * (int64_t)c * ldc;
    for (int r = threadIdx.x; r < m; r += 256) {
      double* z = base + 2 * r;
      if (br == 0.0 && bi == 0.0) {
        z[0] = 0.0;
        z[1] = 0.0;
      } else {
        const double cr = z[0], ci = z[1];
        z[0] = br * cr - bi * ci;
        z[1] = br * ci + bi * cr;
      }
    }
  }
}

template <int TA, int TB, int BN>
static hipError_t launch_tiles(const ZUniformArgs& a, hipStream_t s) {
  const int tiles_m = (a.m + BM - 1) / BM, tiles_n = (a.n + BN - 1) / BN;
  const int64_t tpi = (int64_t)tiles_m * tiles_n;
  return launch_in_parts(tpi, a.batch, BN * 4, [&](int64_t b0, int64_t total, int64_t per_xcd,
                                                   dim3 grid) {
    hipLaunchKernelGGL((k_uniform_z<TA, TB, BN>), grid, dim3(BN * 4), 0, s, a.m, a.n, a.k,
                       a.alpha[0], a.alpha[1], a.A + b0, a.lda, a.B + b0, a.ldb, a.beta[0],
                       a.beta[1], a.C + b0, a.ldc, tiles_m, (int)tpi, total, per_xcd);
    return hipGetLastError();
  });
}

// Tile width.  64 columns are the fastest where they are all C's (2,000 x 256^3:
// 4.04 ms, 32 columns 4.39, 16 5.32), so 32 are taken where they leave a tenth
// or more less padding: n = 24 (5,000 x 200 x 24 x 300) 2.01 -> 1.71 ms, n = 96
// (5,000 x 200 x 96 x 100) 2.16 -> 1.89, n = 160 (2,000 x 256 x 160 x 200) 2.33 ->
// 2.21.  16 only for n <= 16: 5,000 x 200 x 16 x 300 1.29 ms with 32, 1.20 with 16,
// but n = 48 1.25 with 16 and 1.18 with 64.
template <int TA, int TB>
static hipError_t launch(const ZUniformArgs& a, hipStream_t s) {
  if (a.n <= 16) return launch_tiles<TA, TB, 16>(a, s);
  const int64_t w32 = ((int64_t)a.n + 31) / 32 * 32, w64 = ((int64_t)a.n + 63) / 64 * 64;
  return 11 * w32 < 10 * w64 ? launch_tiles<TA, TB, 32>(a, s) : launch_tiles<TA, TB, 64>(a, s);
}

}  // namespace cplx

hipError_t launch_zgemm(const ZUniformArgs& a, hipStream_t s) {
  using namespace cplx;
  switch (a.ta * 3 + a.tb) {
    case 0: return launch<0, 0>(a, s);
    case 1: return launch<0, 1>(a, s);
    case 2: return launch<0, 2>(a, s);
    case 3: return launch<1, 0>(a, s);
    case 4: return launch<1, 1>(a, s);
    case 5: return launch<1, 2>(a, s);
    case 6: return launch<2, 0>(a, s);
    case 7: return launch<2, 1>(a, s);
    default: return launch<2, 2>(a, s);
  }
}

hipError_t launch_zscale(const double* beta, double* const* C, int64_t ldc, int m, int n,
                         int batch, hipStream_t s) {
  const int64_t cols = (int64_t)n * batch;
  if (cols <= 0) return hipSuccess;
  const int64_t grid = cols < 65536 ? cols : 65536;
  hipLaunchKernelGGL(cplx::k_zscale, dim3((unsigned)grid), dim3(256), 0, s, beta[0], beta[1], C,
                     ldc, m, n, cols);
  return hipGetLastError();
}

}  // namespace bg
