// Batched FP64 GEMM kernels for CDNA4 (gfx950).
//
// Operation (the paper, Section II, Eq. 1): for every instance i,
//   C_i <- alpha * op(A_i) * op(B_i) + beta * C_i,   column-major, FP64.
// The paper builds each product from a 2-D grid of C tiles, one thread block
// per tile (Section II); here one workgroup computes one C tile on the FP64
// matrix cores, operands staged through LDS.
//
// Matrix-core instruction.  v_mfma_f64_4x4x4_4b_f64 performs four independent
// 4x4x4 products per wave (blocks b = 0..3).  Lane 16 s + 4 b + i holds
// element (i, s) of block b's first operand, lane 16 s + 4 b + j holds element
// (s, j) of its second operand, and the result element (i, j) of block b lands
// in lane 16 i + 4 b + j (checked on the device by the lane-layout test).  On
// gfx950 this instruction sustains about 1.5x the FP64 rate of the 16x16x4
// form, so the tiles are built from it.
//
// Roles.  Of the two operands of the product, one -- "P" -- is read as a
// 16-row slab: lane 16 s + r holds P(p0 + r, k_s), so the four blocks cover
// 16 consecutive P indices.  The other -- "Q" -- is read replicated: lane
// 16 s + 4 b + j holds Q(q0 + j, k_s) for every b.  One instruction then
// yields a 16 x 4 block of P x Q^T: lane 16 i + 4 b + j holds the sum over s
// of P(p0 + 4 b + i, k_s) Q(q0 + j, k_s).  P is op(A) and Q is op(B)^T, so the
// block is a piece of C whose 16 rows sit in 16 lanes.
//
// Contraction order.  A 16-wide slice of k starting at kk is consumed by four
// instructions t = 0..3; instruction t gives lane group s the index
// k = kk + 2 s + 8 (t / 2) + (t % 2).  Any bijection is valid if both operands
// use it; this one puts each t-pair on adjacent k, so a K-contiguous operand
// feeds two instructions with one 16-byte LDS read.  Every tile class walks k
// in the same slices and order, so a given element of C gets the same bits
// from every class, alone or in any batch.
#include <type_traits>

#include "bgemm_internal.h"
#include "bgemm_tiles.h"

namespace bg {

typedef double d2 __attribute__((ext_vector_type(2)));
// a pair of doubles at any 8-byte boundary: with an odd leading dimension
// every other column's pairs start off a 16-byte boundary, and the memory
// system serves such 16-byte accesses (unaligned access mode)
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// Explicit address spaces: matrices are global memory (address space 1),
// operand tiles are LDS (address space 3).  Without them the compiler falls
// back to flat instructions, which count against both the vector-memory and
// the LDS wait counters and so serialise LDS reads behind global prefetches.
#define AS_GLOBAL __attribute__((address_space(1)))
#define AS_LDS __attribute__((address_space(3)))
typedef const AS_GLOBAL double* gcptr;
typedef AS_GLOBAL double* gptr;

// Nontemporal accesses to C: a tile reads its part of C once and writes it once
// (200,000 x 64^3, half of whose bytes are C, runs 2.5-3.5 % faster with them,
// 256^3 0.1-0.7 %).  Operand loads stay ordinary: the tiles of an instance share
// its panels through the caches.
__device__ __forceinline__ d2 ld_c(const AS_GLOBAL d2u* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void st_c(AS_GLOBAL d2u* p, d2 v) {
  __builtin_nontemporal_store((d2u)v, p);
}

// s_waitcnt immediate: vector-memory count vm, LDS/scalar count lgkm, export
// count unconstrained (gfx9 encoding).
constexpr int waitcnt_imm(int vm, int lgkm) {
  return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm & 15) << 8);
}

// ---------------------------------------------------------------------------
// The tile kernel.  Operand tiles go straight from global memory to LDS in
// 16-byte units (two doubles along the operand's contiguous dimension; a unit
// starts at an 8-byte boundary whenever its column does) and are read back as
// whole units.  P is op(A), Q is op(B)^T, so a 16 x 4 result block is a piece of
// C.
//
// Rows and columns of a wave's tile are dealt to the instructions so that a
// unit is used whole: slabs 2a and 2a + 1 hold the even and the odd ones of
// rows 32a .. 32a + 31, so an MN-contiguous P unit (two rows at one k) feeds
// both, and a lane ends with pairs of adjacent rows of C, 16 lanes on 256
// contiguous bytes of a column: C is read and written 16 bytes at a time
// without a trip through LDS.  An MN-contiguous Q unit feeds two column groups
// the same way.  Which row a lane holds does not enter its sums, whose order
// over k is the one of every class.
//
// What bounds it: the matrix cores, and on them the power budget.  Large waves
// (64 x 64 of the 128 x 128 tile) take 256 matrix-core instructions between
// barriers and read the fewest LDS bytes per instruction; two stages are
// enough because the two or three workgroups a CU holds cover a step's load
// latency.  5,000 x 512^3: matrix cores 0.80 -> 0.88 busy, 23.0 -> 20.9 ms (58.4
// -> 64.2 TFLOP/s, at a clock that drops as they fill); 20,000 x 256^3 13.1 ->
// 12.0 ms, against eight waves of 16 x 64 on a 128 x 64 tile with three stages;
// 3,000 x 129 x 513 x 257 transposed 3.95 -> 2.91 ms with the finer tiles, 100,000 x
// 16^3 0.54 -> 0.23 against staging through registers.
// 128 x 64 tiles of four 64 x 32 waves: 21.6 / 12.1 ms; 64 x 128: as 128 x 64;
// 64 x 64 of 64 x 16 waves: 23.8 / 13.3 (with a slower clock, the others 23.0 /
// 13.0); three stages of it 24.1 / 13.6; the refill right after the barrier
// +1.5 %; Q groups eight, four or two at a time within 1 %, two need the fewest
// registers.
//
// LDS layout (units).  A K-contiguous operand has rows of 8 units: row mn sits
// at rho(mn) (its two low bits swapped), unit u at u ^ f(mn).  An MN-contiguous
// one has a row per k; a Q tile's units sit at u ^ 4 in every other pair of
// rows.  With these every fragment read is free of bank conflicts (a 16-byte
// read is served sixteen lanes at a time, eight from each of two lane groups);
// with f = mn / 2 and rho, f trivial on Q, 40 % of the LDS's cycles were.
// ---------------------------------------------------------------------------
typedef AS_LDS d2* uptr;
typedef const AS_LDS d2* ucptr;

// `once`: C's lines are not shared with other tiles' if its columns are whole
// 128-byte lines (then C is touched nontemporally on interior tiles).
template <class CF, bool TA, bool TB>
__device__ __forceinline__ void pipe_tile(const double* A_, int64_t lda, const double* B_,
                                          int64_t ldb, double* C_, int64_t ldc, int M, int N, int K,
                                          double alpha, double beta, int m0, int n0, uptr lds,
                                          bool once) {
  const gcptr A = (gcptr)A_;
  const gcptr B = (gcptr)B_;
  const gptr C = (gptr)C_;
  constexpr bool AK = TA, BKC = !TB;   // K-contiguous operands
  using At = PTile<CF::BM, CF::BK, AK, true>;
  using Bt = PTile<CF::BN, CF::BK, BKC, false>;
  constexpr int FP = CF::FP, GQ = CF::GQ, NW = CF::NW, BK = CF::BK;
  constexpr int A_UNITS = CF::BM * BK / 2;
  int tid;
  // opaque, so that lane-dependent offsets are not kept live across a
  // persistent caller's tiles
  asm volatile("v_mov_b32 %0, %1" : "=v"(tid) : "v"((int)threadIdx.x));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = CF::wave_row(wave), wn0 = CF::wave_col(wave);
  const bool use_product = !(alpha == 0.0 || K == 0);

  double acc[FP][GQ];
#pragma unroll
  for (int i = 0; i < FP; ++i)
#pragma unroll
    for (int j = 0; j < GQ; ++j) acc[i][j] = 0.0;

  if (use_product) {
    // This thread's units of a stage.  Units whose row or column lies outside
    // the matrix re-read the tile's first one: in bounds, every wave issues the
    // same number of direct loads (the stage waits count them), and their
    // products only reach C elements outside C.  A pair straddling an odd
    // extent reads the element after it (padding, or the next column), except
    // in the last step of such a tile, which goes through registers.
    // An MN-contiguous operand's units lie a fixed number of k rows apart when
    // the waves' chunks are whole rows and no chunk is loaded twice: one pointer
    // then serves them all.
    constexpr bool STEP_A = !AK && NW * 64 % At::UR == 0 && CF::CA % NW == 0;
    constexpr bool STEP_B = !BKC && NW * 64 % Bt::UR == 0 && CF::CB % NW == 0;
    static_assert(!STEP_B || NW * 64 / Bt::UR % 4 == 0, "whole turns of the Q swizzle apart");
    constexpr int QA = STEP_A ? 1 : CF::PA, QB = STEP_B ? 1 : CF::PB;
    gcptr pa[QA], pb[QB];
#pragma unroll
    for (int i = 0; i < QA; ++i) {
      int mn, k;
      At::at((i * NW + wave) % CF::CA * 64 + lane, mn, k);
      const int r = m0 + mn < M ? m0 + mn : m0;
      pa[i] = A + (AK ? (int64_t)r * lda + k : (int64_t)k * lda + r);
    }
#pragma unroll
    for (int i = 0; i < QB; ++i) {
      int mn, k;
      Bt::at((i * NW + wave) % CF::CB * 64 + lane, mn, k);
      const int c = n0 + mn < N ? n0 + mn : n0;
      pb[i] = B + (BKC ? (int64_t)c * ldb + k : (int64_t)k * ldb + c);
    }
    auto a_at = [&](int i) {
      return STEP_A ? pa[0] + i * (NW * 64 / At::UR) * lda : pa[STEP_A ? 0 : i];
    };
    auto b_at = [&](int i) {
      return STEP_B ? pb[0] + i * (NW * 64 / Bt::UR) * ldb : pb[STEP_B ? 0 : i];
    };
    const int64_t sa = AK ? BK : BK * lda, sb = BKC ? BK : BK * ldb;
    const int nk = (K + BK - 1) / BK;
    const bool a_odd = !AK && (M & 1) && m0 + CF::BM > M;
    const bool b_odd = !BKC && (N & 1) && n0 + CF::BN > N;
    const bool tail = (K % BK != 0) || a_odd || b_odd;

    // one unit of the last step through registers, zero beyond K; addresses
    // clamped into the matrix, so every load is unconditional
    auto tail_unit = [&](gcptr p, int64_t ld, bool kc, int mn, int ext, int k) -> d2 {
      const int over = k >= K ? k - (K - 1) : 0;
      if (kc) {
        const double x = p[-over], y = p[k + 1 < K ? 1 : -over];
        return d2{k < K ? x : 0.0, k + 1 < K ? y : 0.0};
      }
      p -= over * ld;
      const double x = p[0], y = p[mn + 1 < ext ? 1 : 0];
      return d2{over ? 0.0 : x, over ? 0.0 : y};
    };
    auto issue = [&](int kt, int st) {
      const uptr la = lds + st * CF::STAGE, lb = la + A_UNITS;
      if (kt == nk - 1 && tail) {
        const int k0 = kt * BK;
#pragma unroll
        for (int i = 0; i < CF::PA; ++i) {
          int mn, k;
          const int p = (i * NW + wave) % CF::CA * 64 + lane;
          At::at(p, mn, k);
          const int r = m0 + mn < M ? m0 + mn : m0;
          la[p] = tail_unit(a_at(i), lda, AK, r, M, k0 + k);
        }
#pragma unroll
        for (int i = 0; i < CF::PB; ++i) {
          int mn, k;
          const int p = (i * NW + wave) % CF::CB * 64 + lane;
          Bt::at(p, mn, k);
          const int c = n0 + mn < N ? n0 + mn : n0;
          lb[p] = tail_unit(b_at(i), ldb, BKC, c, N, k0 + k);
        }
      } else {
#pragma unroll
        for (int i = 0; i < CF::PA; ++i)
          __builtin_amdgcn_global_load_lds((const AS_GLOBAL void*)a_at(i),
                                           (AS_LDS void*)(la + (i * NW + wave) % CF::CA * 64), 16,
                                           0, 0);
#pragma unroll
        for (int i = 0; i < CF::PB; ++i)
          __builtin_amdgcn_global_load_lds((const AS_GLOBAL void*)b_at(i),
                                           (AS_LDS void*)(lb + (i * NW + wave) % CF::CB * 64), 16,
                                           0, 0);
#pragma unroll
        for (int i = 0; i < QA; ++i) pa[i] += sa;
#pragma unroll
        for (int i = 0; i < QB; ++i) pb[i] += sb;
      }
    };
    issue(0, 0);

    // lane addresses of the fragment reads; everything else is a constant offset
    int ap[At::BASES], bp[Bt::BASES];
#pragma unroll
    for (int v = 0; v < At::BASES; ++v) ap[v] = At::p_base(wm0, lane, v);
#pragma unroll
    for (int v = 0; v < Bt::BASES; ++v) bp[v] = A_UNITS + Bt::q_base(wn0, lane, v);

    // Step kt lives in stage kt mod 2.  Its loads were issued a step ago; the
    // wait and the barrier publish every wave's part, and only after it is the
    // other stage, read one step earlier, refilled.  NPA of the wave's slabs and
    // GQA of its column groups take part (fewer on edge tiles, none for a wave
    // outside C); every wave reaches the same barriers.
    auto step = [&](int kt, auto stage_c, auto npa_c, auto gqa_c) {
      constexpr int st = decltype(stage_c)::value;
      constexpr int NPA = decltype(npa_c)::value, GQA = decltype(gqa_c)::value;
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_setprio(1);
      auto refill = [&]() {
        asm volatile("" ::: "memory");
        if (kt + 1 < nk) issue(kt + 1, st ^ 1);
        asm volatile("" ::: "memory");
      };
      if constexpr (NPA == 0) refill();
      const ucptr stage = lds + st * CF::STAGE;
      if constexpr (NPA > 0) {
#pragma unroll
        for (int tp = 0; tp < 2; ++tp) {
          double fp[NPA][2];
#pragma unroll
          for (int a = 0; a < NPA / 2; ++a)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const d2 x = stage[ap[AK ? 2 * tp + u : 0] + At::p_offset(tp, u, a)];
              if constexpr (AK) { fp[2 * a + u][0] = x.x; fp[2 * a + u][1] = x.y; }
              else { fp[2 * a][u] = x.x; fp[2 * a + 1][u] = x.y; }
            }
          // Q groups two at a time: more live fragments would cost the
          // registers of a resident workgroup
#pragma unroll
          for (int h = 0; h < GQA; h += 2) {
            double fq[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const d2 x = stage[bp[BKC ? 0 : (h / 2) & 1] + Bt::q_offset(tp, u, h)];
              if constexpr (BKC) { fq[u][0] = x.x; fq[u][1] = x.y; }
              else { fq[0][u] = x.x; fq[1][u] = x.y; }
            }
            if (tp == 1 && h == 0) refill();
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int i = 0; i < NPA; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                  acc[i][h + j] = __builtin_amdgcn_mfma_f64_4x4x4f64(fp[i][u], fq[j][u],
                                                                     acc[i][h + j], 0, 0, 0);
          }
        }
      }
      __builtin_amdgcn_s_setprio(0);
    };
    auto kloop = [&](auto npa_c, auto gqa_c) {
      for (int kt = 0; kt < nk; kt += 2) {
        step(kt, std::integral_constant<int, 0>{}, npa_c, gqa_c);
        if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>{}, npa_c, gqa_c);
      }
    };
    using std::integral_constant;
    const int pairs = n0 + wn0 < N ? (M - m0 - wm0 + 31) / 32 : 0;
    // (on the 64-row waves of a transposed A the registers do not allow it)
    const bool half = !(AK && FP == 4) && n0 + wn0 + CF::WN / 2 >= N;
    auto columns = [&](auto npa_c) {
      if (half) kloop(npa_c, integral_constant<int, GQ / 2>{});
      else kloop(npa_c, integral_constant<int, GQ>{});
    };
    if (pairs >= FP / 2) columns(integral_constant<int, FP>{});
    else if (FP > 2 && pairs == 1) columns(integral_constant<int, 2>{});
    else kloop(integral_constant<int, 0>{}, integral_constant<int, GQ>{});
  }

  // Epilogue.  Lane 16 i + 4 b + j holds rows r0 + 32 a and the next (slabs 2a,
  // 2a + 1) and one column per group.  C is read (beta != 0) GE groups at a
  // time before their stores.
  if (!use_product && beta == 1.0) return;
  int le;   // the lane again, not kept in a register through the k loop
  asm volatile("v_and_b32 %0, 63, %1" : "=v"(le) : "v"((int)threadIdx.x));
  const int r0 = m0 + CF::lane_row(wm0, le);
  auto c_col = [&](int g) { return n0 + CF::lane_col(BKC, wn0, le, g); };
  constexpr int GE = CF::GE;
  auto combine = [&](int a, int g, d2 c) {
    // alpha acc is rounded, beta c fused: written out, since the compiler may
    // contract the plain sum either way and every class must round alike
    d2 y{alpha * acc[2 * a][g], alpha * acc[2 * a + 1][g]};
    if (beta != 0.0) y = d2{__builtin_fma(beta, c.x, y.x), __builtin_fma(beta, c.y, y.y)};
    return y;
  };
  auto interior = [&](auto stream_c) {
    constexpr bool STREAM = decltype(stream_c)::value;
#pragma unroll
    for (int g0 = 0; g0 < GQ; g0 += GE) {
      d2 cv[FP / 2][GE];
      if (beta != 0.0) {
#pragma unroll
        for (int g = 0; g < GE; ++g)
#pragma unroll
          for (int a = 0; a < FP / 2; ++a) {
            const auto p = (const AS_GLOBAL d2u*)(C + r0 + (int64_t)c_col(g0 + g) * ldc + 32 * a);
            if constexpr (STREAM) cv[a][g] = ld_c(p);
            else cv[a][g] = *p;
          }
      }
#pragma unroll
      for (int g = 0; g < GE; ++g)
#pragma unroll
        for (int a = 0; a < FP / 2; ++a) {
          const auto p = (AS_GLOBAL d2u*)(C + r0 + (int64_t)c_col(g0 + g) * ldc + 32 * a);
          const d2 y = combine(a, g0 + g, cv[a][g]);
          if constexpr (STREAM) st_c(p, y);
          else *p = y;
        }
    }
  };
  if (use_product && m0 + CF::BM <= M && n0 + CF::BN <= N) {
    // Nontemporal where every line of C belongs to this tile alone; a line cut
    // between two accesses is better merged in L2 (the variable-size batch ran
    // 2 % slower, its short-k tiles 20 %, with nontemporal partial lines).
    if (once && (((uintptr_t)C_ | (uintptr_t)(8 * ldc)) & 127) == 0) interior(std::true_type{});
    else interior(std::false_type{});
    return;
  }
  constexpr int GB = CF::GB;   // edge tiles: bounds take registers too
#pragma unroll
  for (int g0 = 0; g0 < GQ; g0 += GB) {
    d2 cv[FP / 2][GB];
#pragma unroll
    for (int g = 0; g < GB; ++g)
#pragma unroll
      for (int a = 0; a < FP / 2; ++a) {
        cv[a][g] = d2{0.0, 0.0};
        const int r = r0 + 32 * a, c = c_col(g0 + g);
        if (beta != 0.0 && c < N && r < M) {
          const gcptr p = (gcptr)C + r + (int64_t)c * ldc;
          if (r + 1 < M) cv[a][g] = *(const AS_GLOBAL d2u*)p;
          else cv[a][g].x = p[0];
        }
      }
#pragma unroll
    for (int g = 0; g < GB; ++g)
#pragma unroll
      for (int a = 0; a < FP / 2; ++a) {
        const int r = r0 + 32 * a, c = c_col(g0 + g);
        if (c >= N || r >= M) continue;
        d2 y;
        if (use_product) y = combine(a, g0 + g, cv[a][g]);
        else y = beta == 0.0 ? d2{0.0, 0.0} : d2{beta * cv[a][g].x, beta * cv[a][g].y};
        const gptr p = C + r + (int64_t)c * ldc;
        if (r + 1 < M) *(AS_GLOBAL d2u*)p = y;
        else p[0] = y.x;
      }
  }
}

// ---------------------------------------------------------------------------
// Uniform batch: one workgroup per (instance, C tile).  Workgroups are handed
// to the eight XCDs round-robin by id, so id -> (instance, tile) is remapped
// to give each XCD a contiguous range of tiles: all tiles of an instance run
// on one XCD at about the same time and share its L2 for the A/B panels.
// ---------------------------------------------------------------------------
constexpr int NUM_XCD = 8;

template <class CF, bool TA, bool TB>
__global__ __launch_bounds__(CF::NT, CF::WAVES) void k_uniform(
    int M, int N, int K, double alpha, const double* const* __restrict__ Ap, int64_t lda,
    const double* const* __restrict__ Bp, int64_t ldb, double beta,
    double* const* __restrict__ Cp, int64_t ldc, int tiles_m, int tiles_per_inst,
    int64_t total_tiles, int64_t per_xcd) {
  __shared__ __align__(16) double lds[CF::LDS];
  const int64_t bid = blockIdx.x;
  const int64_t id = (bid % NUM_XCD) * per_xcd + bid / NUM_XCD;
  if (id >= total_tiles) return;
  const int64_t inst = id / tiles_per_inst;
  const int t = (int)(id - inst * tiles_per_inst);
  pipe_tile<CF, TA, TB>(Ap[inst], lda, Bp[inst], ldb, Cp[inst], ldc, M, N, K, alpha, beta,
                        t % tiles_m * CF::BM, t / tiles_m * CF::BN, (uptr)lds, true);
}

template <class CF, bool TA, bool TB>
static hipError_t launch_uniform_t(const UniformArgs& a, hipStream_t s) {
  const int tiles_m = (a.m + CF::BM - 1) / CF::BM;
  const int tiles_n = (a.n + CF::BN - 1) / CF::BN;
  const int64_t tpi = (int64_t)tiles_m * tiles_n;
  return launch_in_parts(tpi, a.batch, CF::NT, [&](int64_t b0, int64_t total, int64_t per_xcd,
                                                   dim3 grid) {
    hipLaunchKernelGGL((k_uniform<CF, TA, TB>), grid, dim3(CF::NT), 0, s, a.m, a.n, a.k, a.alpha,
                       a.A + b0, a.lda, a.B + b0, a.ldb, a.beta, a.C + b0, a.ldc, tiles_m, (int)tpi,
                       total, per_xcd);
    return hipGetLastError();
  });
}

template <class CF>
static hipError_t launch_uniform_c(const UniformArgs& a, hipStream_t s) {
  if (!a.ta && !a.tb) return launch_uniform_t<CF, false, false>(a, s);
  if (!a.ta && a.tb) return launch_uniform_t<CF, false, true>(a, s);
  if (a.ta && !a.tb) return launch_uniform_t<CF, true, false>(a, s);
  return launch_uniform_t<CF, true, true>(a, s);
}

// Tile of a uniform batch: the one with the least estimated time.  Per C element
// and k a tile takes `weight`, and `fixed` k more for its first loads and its C.
// Of the area, what the matrix-core instructions of edge waves skip counts by
// PADDED only (its loads and its slot remain).  All of it is fitted to the times
// of every shape on 1,285 batches, m, n, k in 7..513, whole and ragged, every
// operand layout, with and without C and padding, two thirds of them streaming
// from HBM and the others down to a few hundred instances (which stay in the
// caches, so that padding costs more): the choice is 1.0 % from the best shape on
// average there, 1.9 % on 200 batches that were not fitted.  Times in us of the
// shapes in the table's order, the choice first:
//   20,000 x 256^3      11,990 | 11,990 12,140 13,700 12,660 13,490 13,490 14,710 17,020
//   1,000 x 512^3        4,204 |  4,204  4,314  4,604  4,465  4,778  4,768  5,196  5,824
//   60,000 x 128^3       5,821 |  5,805  5,821  6,676  6,016  6,445  6,485  7,050  8,274
//   15,000 x 256 x 144 x 80  2,497 | 3,683 2,669 2,497 2,676 2,719 2,945 3,048 3,439
//   60,000 x 128 x 48 x 64   1,927 | 3,188 2,172 1,927 2,082 2,018 2,095 2,157 2,244
// A single 64 x 64 tile with neither operand transposed is bound by memory at
// short k and prefers two half tiles in flight: 64 x 32 against 64 x 64 is 2.5 %
// faster on 68 sizes of k <= 32, at k of 33 to 64 1.2 % faster on 16 with both
// extents above 48 (200,000 x 64^3 4.40 against 4.44 ms) and 2.4 % slower on 16
// others; with a transposed operand it is 4.6 % slower on 26 of k <= 32.  A batch
// that would not give every CU `need` tiles of a shape goes to a finer one: a
// short batch is latency-bound, and more, shorter tiles finish sooner (1 x 512^3
// 22.1 us on 64 x 64, 14.7 on 64 x 32 and 14.2 on 32 x 32 tiles; 7 x 512^3 37.5 / 38.2
// / 38.3, and 70 on 128 x 128).
struct TileChoice {
  TileClass cls;
  int bm, bn, wn;
  double weight, fixed, need;
};
static constexpr TileChoice kTiles[] = {
    {TC_128, 128, 128, 64, 1.000, 14, 2},    {TC_128x64, 128, 64, 32, 1.026, 7.5, 2},
    {TC_128x48, 128, 48, 48, 1.137, 8, 2},   {TC_64, 64, 64, 32, 1.138, 4, 1},
    {TC_64x32, 64, 32, 16, 1.239, 3, .5},    {TC_32x64, 32, 64, 16, 1.178, 6, .5},
    {TC_32, 32, 32, 16, 1.459, 5.5, 0},      {TC_32x16, 32, 16, 16, 1.729, 14.5, 0},
};
constexpr double PADDED = 0.75;

TileClass pick_uniform_class(bool nn, int m, int n, int k, int batch, int num_cus, int force) {
  if (force >= 0 && force < TC_SHAPES) return (TileClass)force;
  auto up = [](int x, int to) { return (double)((x + to - 1) / to) * to; };
  const double k16 = up(k, 16);
  const bool halves = nn && m > 32 && m <= 64 && n > 32 && n <= 64 &&
                      k <= (m > 48 && n > 48 ? 64 : 32);
  TileClass best = TC_128;   // the coarsest, should every grid be too large
  double least = 0.0;
  // unrolled: the sizes are constants, so no division is left (49 ns a call)
#pragma unroll
  for (const TileChoice& t : kTiles) {
    const double area = up(m, t.bm) * up(n, t.bn);
    const double tiles = area * (1.0 / (t.bm * t.bn));
    if (tiles * batch < t.need * num_cus || tiles * batch > INT32_MAX - 8) continue;
    const double used = up(m, 32) * up(n, t.wn / 2);
    double cost = t.weight * k16 * (PADDED * area + (1 - PADDED) * used) + t.fixed * area;
    if (t.cls == TC_64x32 && halves) cost *= 0.85;
    if (least == 0.0 || cost < least) {
      least = cost;
      best = t.cls;
    }
  }
  return best;
}

hipError_t launch_uniform(const UniformArgs& a, TileClass cls, hipStream_t s) {
  switch (cls) {
    case TC_32: return launch_uniform_c<P32>(a, s);
    case TC_64: return launch_uniform_c<P64>(a, s);
    case TC_128x64: return launch_uniform_c<P128x64>(a, s);
    case TC_64x32: return launch_uniform_c<P64x32>(a, s);
    case TC_128x48: return launch_uniform_c<P128x48>(a, s);
    case TC_32x64: return launch_uniform_c<P32x64>(a, s);
    case TC_32x16: return launch_uniform_c<P32x16>(a, s);
    default: return launch_uniform_c<P128>(a, s);
  }
}

// ---------------------------------------------------------------------------
// Several short batches of square products in one launch (the request loop's
// tick: one batch per client size).  Launched one after another each of them
// leaves most of the chip idle and waits for its own slowest tile; here the
// tiles of all of them are in flight together, largest matrices first.  Each
// batch's tiles are dealt to the XCDs in contiguous ranges, as in k_uniform.
// What bounds it is the largest matrices' k loop on the CUs that hold two of
// their tiles.  Measured on a tick of 32 clients (sizes 32..512, seven of
// 512): five launches 92 us, one 47 (43 on the present tile); draining 2,000
// requests of 1..16 products 86 -> 52 -> 47 ms.
// ---------------------------------------------------------------------------
constexpr int MAX_GROUPS = 16;

struct GroupTable {
  int count;
  int n[MAX_GROUPS];
  int tiles[MAX_GROUPS];          // C tiles of the batch
  int slot[MAX_GROUPS + 1];       // first workgroup of the batch on each XCD
  const double* const* A[MAX_GROUPS];
  const double* const* B[MAX_GROUPS];
  double* const* C[MAX_GROUPS];
};

template <class CF>
__global__ __launch_bounds__(CF::NT, CF::WAVES) void k_uniform_groups(GroupTable gt) {
  __shared__ __align__(16) double lds[CF::LDS];
  const int x = blockIdx.x % NUM_XCD, slot = blockIdx.x / NUM_XCD;
  int g = 0;
  while (g + 1 < gt.count && slot >= gt.slot[g + 1]) ++g;
  const int id = x * (gt.slot[g + 1] - gt.slot[g]) + slot - gt.slot[g];
  if (id >= gt.tiles[g]) return;
  const int n = gt.n[g];
  const int tiles_m = (n + CF::BM - 1) / CF::BM, tpi = tiles_m * ((n + CF::BN - 1) / CF::BN);
  const int inst = id / tpi, t = id - inst * tpi;
  pipe_tile<CF, false, false>(gt.A[g][inst], n, gt.B[g][inst], n, gt.C[g][inst], n, n, n, n, 1.0,
                              0.0, t % tiles_m * CF::BM, t / tiles_m * CF::BN, (uptr)lds, true);
}

template <class CF>
static hipError_t launch_groups(const GroupTable& gt, hipStream_t s) {
  hipLaunchKernelGGL((k_uniform_groups<CF>), dim3((unsigned)(gt.slot[gt.count] * NUM_XCD)),
                     dim3(CF::NT), 0, s, gt);
  return hipGetLastError();
}

hipError_t launch_square_groups(const SquareGroup* groups, int count, int num_cus, hipStream_t s) {
  auto fills_chip = [&](const SquareGroup& q) {
    return (int64_t)((q.n + 127) / 128) * ((q.n + 63) / 64) * q.batch >= 2 * (int64_t)num_cus;
  };
  int64_t tiles64 = 0;
  for (int i = 0; i < count; ++i) {
    const SquareGroup& q = groups[i];
    if (!fills_chip(q)) {
      tiles64 += (int64_t)((q.n + 63) / 64) * ((q.n + 63) / 64) * q.batch;
      continue;
    }
    UniformArgs a;
    a.ta = a.tb = false;
    a.m = a.n = a.k = q.n;
    a.alpha = 1.0; a.beta = 0.0;
    a.A = q.A; a.lda = q.n; a.B = q.B; a.ldb = q.n; a.C = q.C; a.ldc = q.n;
    a.batch = q.batch;
    const hipError_t e =
        launch_uniform(a, pick_uniform_class(true, q.n, q.n, q.n, q.batch, num_cus, -1), s);
    if (e != hipSuccess) return e;
  }
  // the short ones, MAX_GROUPS to a launch; tile shapes as for one short batch
  const bool narrow = tiles64 <= num_cus;
  GroupTable gt;
  gt.count = 0;
  gt.slot[0] = 0;
  for (int i = 0; i < count; ++i) {
    const SquareGroup& q = groups[i];
    if (fills_chip(q)) continue;
    const int g = gt.count++;
    gt.n[g] = q.n;
    gt.tiles[g] = ((q.n + 63) / 64) * ((q.n + (narrow ? 31 : 63)) / (narrow ? 32 : 64)) * q.batch;
    gt.slot[g + 1] = gt.slot[g] + (gt.tiles[g] + NUM_XCD - 1) / NUM_XCD;
    gt.A[g] = q.A; gt.B[g] = q.B; gt.C[g] = q.C;
    if (gt.count == MAX_GROUPS) {
      const hipError_t e = narrow ? launch_groups<P64x32>(gt, s) : launch_groups<P64>(gt, s);
      if (e != hipSuccess) return e;
      gt.count = 0;
    }
  }
  if (gt.count == 0) return hipSuccess;
  return narrow ? launch_groups<P64x32>(gt, s) : launch_groups<P64>(gt, s);
}

// C_i <- beta * C_i, or exactly 0 when beta == 0 (C not read).
__global__ __launch_bounds__(256) void k_scale(double beta, double* const* __restrict__ Cp,
                                               int64_t ldc, int m, int n, int64_t total_cols) {
  for (int64_t col = blockIdx.x; col < total_cols; col += gridDim.x) {
    const int64_t inst = col / n;
    const int j = (int)(col - inst * n);
    double* p = Cp[inst] + (int64_t)j * ldc;
    for (int r = threadIdx.x; r < m; r += blockDim.x) p[r] = (beta == 0.0) ? 0.0 : beta * p[r];
  }
}

hipError_t launch_scale(double beta, double* const* C, int64_t ldc, int m, int n, int batch,
                        hipStream_t s) {
  const int64_t cols = (int64_t)n * batch;
  const int64_t grid = cols < 65536 ? cols : 65536;
  hipLaunchKernelGGL(k_scale, dim3((unsigned)grid), dim3(256), 0, s, beta, C, ldc, m, n, cols);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Variable-size batch (the paper, Section II: each GEMM gets its own 2-D grid
// of tiles, sizes differ per instance).  Sizes live on the device, so the
// whole plan is made there.  Each instance is assigned one of three tile
// classes (128 x 64, 64 x 64, 32 x 32) by the padded work its C grid costs
// (100,000 mixed sizes 18.5 -> 18.0 ms against register-staged 64 x 64 and 32 x 32
// classes and a 128 x 64 one of eight waves; batches of 500-15,000 with sizes
// from 8..512 2-22 % faster);
// each class gets its own tile queue, and a persistent kernel per class, in
// decreasing tile size, pops tiles from it:
//   1. k_vb_count: validate each instance (info), choose its class, count its
//      C tiles, and scan the counts of each class within blocks of 256;
//   2. k_vb_blocks: scan the block totals of each class (one workgroup),
//      reset the queues;
//   3. k_vb_finish: per-class exclusive prefix P_c[i] over instances;
//   4. k_vb_map: when it fits in the workspace, a map tile -> instance;
//   5. k_vb_exec (x3): a persistent grid per class; each workgroup pops tile
//      numbers from its class's atomic counters until the queue is empty.
// ---------------------------------------------------------------------------
#ifndef BG_CFGVB_L
#define BG_CFGVB_L 128, 64, 64, 32
#endif
#ifndef BG_CFGVB_M
#define BG_CFGVB_M 64, 64, 32, 32
#endif
#ifndef BG_CFGVB_S
#define BG_CFGVB_S 32, 32, 32, 16
#endif
// Relative cost per padded C element of the three classes, for the choice.  1 :
// 1.1 : 1.3 and 1 : 1.05 : 1.13 (the tiles' rates on whole tiles) ran the 100,000
// mixed sizes 1 and 3 % slower: a persistent workgroup pays for each tile's pop
// and sizes too.
#ifndef BG_VB_WEIGHTS
#define BG_VB_WEIGHTS 1.0f, 1.3f, 2.0f
#endif
using CfgVbL = PCfg<BG_CFGVB_L>;
using CfgVbM = PCfg<BG_CFGVB_M>;
using CfgVbS = PCfg<BG_CFGVB_S>;
constexpr int VB_NC = 3;
constexpr int PLAN_BLOCK = 256;
// Queue heads, one per (class, XCD), each on its own 4 KB line: every pop
// is a device-scope atomic, performed at the memory side, and heads sharing
// a line would serialise all pops of the device on one channel.
#ifndef BG_VB_HEAD_STRIDE
#define BG_VB_HEAD_STRIDE 512
#endif
constexpr int HEAD_STRIDE = BG_VB_HEAD_STRIDE;             // int64 elements
constexpr int HEAD_BASE = HEAD_STRIDE > VB_NC ? HEAD_STRIDE : VB_NC;
constexpr int VB_CTRL = HEAD_BASE + VB_NC * 8 * HEAD_STRIDE;  // totals, then the heads
__device__ __forceinline__ int64_t* vb_head(int64_t* ctrl, int cls, int x) {
  return ctrl + HEAD_BASE + (int64_t)(cls * 8 + x) * HEAD_STRIDE;
}

struct VbLayout {
  int64_t* prefix;   // [VB_NC][batch + 1]
  int64_t* bsum;     // [VB_NC][nblocks]
  int64_t* ctrl;     // [0..2] tiles per class, then the queue heads (vb_head)
  int* map;          // [map_cap]
  int64_t map_cap;
};

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t vbatched_workspace_bytes(int batch) {
  const size_t nb = ((size_t)batch + PLAN_BLOCK - 1) / PLAN_BLOCK;
  return align256(VB_NC * ((size_t)batch + 1) * 8) + align256(VB_NC * nb * 8) +
         align256(VB_CTRL * 8);
}

static VbLayout vb_layout(const VbWorkspace& ws, int batch) {
  VbLayout L;
  char* p = (char*)ws.base;
  const size_t nb = ((size_t)batch + PLAN_BLOCK - 1) / PLAN_BLOCK;
  L.prefix = (int64_t*)p; p += align256(VB_NC * ((size_t)batch + 1) * 8);
  L.bsum = (int64_t*)p; p += align256(VB_NC * nb * 8);
  L.ctrl = (int64_t*)p; p += align256(VB_CTRL * 8);
  const size_t used = (size_t)(p - (char*)ws.base);
  L.map = (int*)p;
  L.map_cap = used < ws.bytes ? (int64_t)((ws.bytes - used) / sizeof(int)) : 0;
  return L;
}

// Argument numbers follow reference-BLAS DGEMM (3 m, 4 n, 5 k, 8 lda, 10 ldb,
// 13 ldc).  Returns 0 for a valid instance.
__device__ __forceinline__ int vb_check(bool ta, bool tb, int m, int n, int k, int lda, int ldb,
                                        int ldc) {
  if (m < 0) return -3;
  if (n < 0) return -4;
  if (k < 0) return -5;
  const int ra = ta ? k : m, rb = tb ? n : k;
  if (lda < (ra > 1 ? ra : 1)) return -8;
  if (ldb < (rb > 1 ? rb : 1)) return -10;
  if (ldc < (m > 1 ? m : 1)) return -13;
  return 0;
}

template <class CF>
__device__ __forceinline__ int64_t vb_tiles(int m, int n) {
  return (int64_t)((m + CF::BM - 1) / CF::BM) * ((n + CF::BN - 1) / CF::BN);
}

// Class with the least weighted padded C area; ties go to the larger tile.
__device__ __forceinline__ int vb_class(int m, int n, int64_t* tiles) {
  const float w[VB_NC] = {BG_VB_WEIGHTS};
  const int64_t t[VB_NC] = {vb_tiles<CfgVbL>(m, n), vb_tiles<CfgVbM>(m, n),
                            vb_tiles<CfgVbS>(m, n)};
  const float area[VB_NC] = {(float)(CfgVbL::BM * CfgVbL::BN), (float)(CfgVbM::BM * CfgVbM::BN),
                             (float)(CfgVbS::BM * CfgVbS::BN)};
  int best = 0;
  float cost = w[0] * area[0] * (float)t[0];
  for (int c = 1; c < VB_NC; ++c) {
    const float x = w[c] * area[c] * (float)t[c];
    if (x < cost) { cost = x; best = c; }
  }
  *tiles = t[best];
  return best;
}

__global__ __launch_bounds__(PLAN_BLOCK) void k_vb_count(
    bool ta, bool tb, const int* __restrict__ m, const int* __restrict__ n,
    const int* __restrict__ k, const int* __restrict__ lda, const int* __restrict__ ldb,
    const int* __restrict__ ldc, double alpha, double beta, int batch, int* __restrict__ info,
    int64_t* __restrict__ prefix, int64_t* __restrict__ bsum) {
  __shared__ int64_t sh[VB_NC][PLAN_BLOCK];
  const int i = blockIdx.x * PLAN_BLOCK + threadIdx.x;
  int64_t tiles = 0;
  int cls = 0;
  if (i < batch) {
    const int mi = m[i], ni = n[i], ki = k[i];
    const int st = vb_check(ta, tb, mi, ni, ki, lda[i], ldb[i], ldc[i]);
    if (info) info[i] = st;
    const bool noop = (alpha == 0.0 || ki == 0) && beta == 1.0;
    if (st == 0 && mi > 0 && ni > 0 && !noop) cls = vb_class(mi, ni, &tiles);
  }
  int64_t mine[VB_NC];
  for (int c = 0; c < VB_NC; ++c) {
    mine[c] = (c == cls) ? tiles : 0;
    sh[c][threadIdx.x] = mine[c];
  }
  __syncthreads();
  for (int off = 1; off < PLAN_BLOCK; off <<= 1) {  // inclusive scans (Hillis-Steele)
    int64_t x[VB_NC];
    for (int c = 0; c < VB_NC; ++c) x[c] = threadIdx.x >= off ? sh[c][threadIdx.x - off] : 0;
    __syncthreads();
    for (int c = 0; c < VB_NC; ++c) sh[c][threadIdx.x] += x[c];
    __syncthreads();
  }
  const int nb = gridDim.x;
  for (int c = 0; c < VB_NC; ++c) {
    if (i < batch) prefix[(int64_t)c * (batch + 1) + i] = sh[c][threadIdx.x] - mine[c];
    if (threadIdx.x == PLAN_BLOCK - 1) bsum[c * nb + blockIdx.x] = sh[c][PLAN_BLOCK - 1];
  }
}

__global__ __launch_bounds__(1024) void k_vb_blocks(int64_t* __restrict__ bsum, int nblocks,
                                                    int64_t* __restrict__ ctrl) {
  // exclusive scan of each class's block sums in place, 1024 per pass
  __shared__ int64_t sh[1024];
  __shared__ int64_t carry;
  for (int c = 0; c < VB_NC; ++c) {
    int64_t* b = bsum + (int64_t)c * nblocks;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nblocks; base += 1024) {
      const int i = base + threadIdx.x;
      const int64_t x = i < nblocks ? b[i] : 0;
      sh[threadIdx.x] = x;
      __syncthreads();
      for (int off = 1; off < 1024; off <<= 1) {
        const int64_t y = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += y;
        __syncthreads();
      }
      if (i < nblocks) b[i] = carry + sh[threadIdx.x] - x;
      __syncthreads();
      if (threadIdx.x == 1023) carry += sh[1023];
      __syncthreads();
    }
    if (threadIdx.x == 0) ctrl[c] = carry;                          // tiles of class c
    if (threadIdx.x < 8) *vb_head(ctrl, c, threadIdx.x) = 0;        // its per-XCD heads
    __syncthreads();
  }
}

__global__ __launch_bounds__(PLAN_BLOCK) void k_vb_finish(int batch, int64_t* __restrict__ prefix,
                                                          const int64_t* __restrict__ bsum,
                                                          const int64_t* __restrict__ ctrl) {
  const int i = blockIdx.x * PLAN_BLOCK + threadIdx.x;
  if (i >= batch) return;
  for (int c = 0; c < VB_NC; ++c) {
    int64_t* pc = prefix + (int64_t)c * (batch + 1);
    pc[i] += bsum[c * gridDim.x + blockIdx.x];
    if (i == batch - 1) pc[batch] = ctrl[c];
  }
}

// Writes the tile -> instance map (class c's tiles at offset sum_{c'<c} T_c')
// once all prefixes are final.
__global__ __launch_bounds__(PLAN_BLOCK) void k_vb_map(int batch, const int64_t* __restrict__ prefix,
                                                       const int64_t* __restrict__ ctrl,
                                                       int* __restrict__ map, int64_t map_cap) {
  int64_t total = 0;
  for (int c = 0; c < VB_NC; ++c) total += ctrl[c];
  if (total > map_cap) return;
  const int i = blockIdx.x * PLAN_BLOCK + threadIdx.x;
  if (i >= batch) return;
  int64_t moff = 0;
  for (int c = 0; c < VB_NC; ++c) {
    const int64_t* pc = prefix + (int64_t)c * (batch + 1);
    const int64_t lo = pc[i], hi = pc[i + 1];
    for (int64_t t = lo; t < hi; ++t) map[moff + t] = i;
    moff += ctrl[c];
  }
}

// A value every lane holds alike, in scalar registers (what is addressed by it
// is then loaded through the scalar cache and stays out of the vector
// registers, which the 128 x 64 tile's budget needs).
__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)(x & 0xffffffff));
  const int hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
  return ((int64_t)hi << 32) | lo;
}

// Instance owning tile q of a class: the last i with P[i] <= q < P[i + 1].
__device__ __forceinline__ int vb_find(const int64_t* __restrict__ prefix, int batch, int64_t q) {
  int lo = 0, hi = batch;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (prefix[mid] <= q) lo = mid; else hi = mid;
  }
  return lo;
}

// The tiles of a class are split into eight equal ranges, one per XCD
// (workgroups reach the XCDs round-robin by id), so that the tiles of an
// instance run on one XCD and share its L2 for the A and B panels.  A
// workgroup pops from its own XCD's range first, then steals from the others
// in turn; every counter is only ever incremented, so each tile is taken
// exactly once and every workgroup leaves after one pass over the eight.
template <class CF, bool TA, bool TB>
__global__ __launch_bounds__(CF::NT, CF::WAVES) void k_vb_exec(
    const int* __restrict__ m, const int* __restrict__ n, const int* __restrict__ k, double alpha,
    const double* const* __restrict__ Ap, const int* __restrict__ lda,
    const double* const* __restrict__ Bp, const int* __restrict__ ldb, double beta,
    double* const* __restrict__ Cp, const int* __restrict__ ldc, int batch, int cls,
    const int64_t* __restrict__ prefix_all, int64_t* __restrict__ ctrl, const int* __restrict__ map,
    int64_t map_cap) {
  __shared__ __align__(16) double lds[CF::LDS];
  __shared__ int64_t s_q;
  const int64_t* prefix = prefix_all + (int64_t)cls * (batch + 1);
  const int64_t total = ctrl[cls];
  if (total == 0) return;   // no tile of this class (uniform across the workgroup)
  int64_t all = 0, moff = 0;
  for (int c = 0; c < VB_NC; ++c) {
    all += ctrl[c];
    if (c < cls) moff += ctrl[c];
  }
  const bool use_map = all <= map_cap;

  const int home = blockIdx.x % NUM_XCD;
  for (int step = 0; step < NUM_XCD; ++step) {
    const int x = (home + step) % NUM_XCD;
    const int64_t lo = total * x / NUM_XCD, hi = total * (x + 1) / NUM_XCD;
    for (;;) {
      if (threadIdx.x == 0)
        s_q = lo + (int64_t)atomicAdd((unsigned long long*)vb_head(ctrl, cls, x), 1ull);
      __syncthreads();
      const int64_t q = uniform64(s_q);
      __syncthreads();
      if (q >= hi) break;
      const int i = use_map ? map[moff + q] : vb_find(prefix, batch, q);
      const int mi = m[i], ni = n[i], ki = k[i];
      const int tiles_m = (mi + CF::BM - 1) / CF::BM;
      const int t = (int)(q - prefix[i]);
      pipe_tile<CF, TA, TB>(Ap[i], lda[i], Bp[i], ldb[i], Cp[i], ldc[i], mi, ni, ki, alpha, beta,
                            t % tiles_m * CF::BM, t / tiles_m * CF::BN, (uptr)lds, false);
      __syncthreads();  // LDS free for the next tile
    }
  }
}

template <class CF, bool TA, bool TB>
static hipError_t launch_vb_exec(const VbatchedArgs& a, const VbLayout& L, int cls, int num_cus,
                                 hipStream_t s) {
  auto kern = k_vb_exec<CF, TA, TB>;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, CF::NT, 0) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  hipLaunchKernelGGL(kern, dim3(num_cus * per_cu), dim3(CF::NT), 0, s, a.m, a.n, a.k, a.alpha,
                     a.A, a.lda, a.B, a.ldb, a.beta, a.C, a.ldc, a.batch, cls, L.prefix, L.ctrl,
                     L.map, L.map_cap);
  return hipGetLastError();
}

template <class CF>
static hipError_t launch_vb_exec_t(const VbatchedArgs& a, const VbLayout& L, int cls, int num_cus,
                                   hipStream_t s) {
  if (!a.ta && !a.tb) return launch_vb_exec<CF, false, false>(a, L, cls, num_cus, s);
  if (!a.ta && a.tb) return launch_vb_exec<CF, false, true>(a, L, cls, num_cus, s);
  if (a.ta && !a.tb) return launch_vb_exec<CF, true, false>(a, L, cls, num_cus, s);
  return launch_vb_exec<CF, true, true>(a, L, cls, num_cus, s);
}

hipError_t launch_vbatched(const VbatchedArgs& a, const VbWorkspace& ws, int num_cus,
                           hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  if (vbatched_workspace_bytes(a.batch) > ws.bytes) return hipErrorOutOfMemory;
  const VbLayout L = vb_layout(ws, a.batch);
  const int nb = (a.batch + PLAN_BLOCK - 1) / PLAN_BLOCK;
  hipLaunchKernelGGL(k_vb_count, dim3(nb), dim3(PLAN_BLOCK), 0, s, a.ta, a.tb, a.m, a.n, a.k, a.lda,
                     a.ldb, a.ldc, a.alpha, a.beta, a.batch, a.info, L.prefix, L.bsum);
  hipLaunchKernelGGL(k_vb_blocks, dim3(1), dim3(1024), 0, s, L.bsum, nb, L.ctrl);
  hipLaunchKernelGGL(k_vb_finish, dim3(nb), dim3(PLAN_BLOCK), 0, s, a.batch, L.prefix, L.bsum,
                     L.ctrl);
  hipLaunchKernelGGL(k_vb_map, dim3(nb), dim3(PLAN_BLOCK), 0, s, a.batch, L.prefix, L.ctrl, L.map,
                     L.map_cap);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = launch_vb_exec_t<CfgVbL>(a, L, 0, num_cus, s)) != hipSuccess) return e;
  if ((e = launch_vb_exec_t<CfgVbM>(a, L, 1, num_cus, s)) != hipSuccess) return e;
  return launch_vb_exec_t<CfgVbS>(a, L, 2, num_cus, s);
}

}  // namespace bg
