// Reduced-precision batched GEMM modes for gfx950 on binary64 inputs and
// outputs (the paper, Section II, Eq. 1, with cheaper inner arithmetic):
//   fp32 : inputs rounded to binary32, products and sums on the binary32
//          matrix cores (v_mfma_f32_16x16x4_f32);
//   bf16 : inputs rounded to binary32 then bfloat16 (nearest even), binary32
//          accumulation (v_mfma_f32_16x16x32_bf16).
// A C entry's sum runs over ascending k, four (fp32) or thirty-two (bf16)
// terms per instruction, zeros appended up to a multiple of 32, whatever the
// tile; so a product's bits do not depend on the tile shape or the batch.
//
// What bounds it: HBM.  At 256^3 the binary64 operands and C are 1.57 MB per
// instance against 33.6 MFLOP, 5.6 ms per 20,000 instances at the 5.6 TB/s
// that streams reach on this card, where the binary32 matrix cores need 4.4
// ms and the bfloat16 ones under 0.5.  So every element is loaded in 16-byte
// pairs, converted once per tile on its way to LDS (4 or 2 bytes instead of
// 8), and the next chunk's loads are in flight in registers during the
// current chunk's products and the other workgroup's conversions; C is
// written once, nontemporally.  Measured on 20,000 x 256^3: fp32 28.5 -> 7.75
// ms, bf16 26.9 -> 5.55 ms (5.6 TB/s) against a kernel that staged binary64
// tiles in LDS behind three barriers per step with no load in flight.
//
// Tile: 128 x 128 or 64 x 64 of C, NT / 64 waves of BM / 2 rows, one 32-wide
// chunk of k per step, two LDS stages, one barrier per step.  The
// instruction's first operand is B's tile and its second A's, so a result
// block is the transpose of a C block and its 16 lanes cover 16 consecutive
// rows of a C column (coalesced epilogue).  Operands must be non-transposed
// (NN).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bgemm_internal.h"

namespace bg {
namespace rounded {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));  // at any 8-byte boundary
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

#define AS_GLOBAL __attribute__((address_space(1)))
typedef const AS_GLOBAL double* gcptr;
typedef AS_GLOBAL double* gptr;

constexpr int BK = 32;

__device__ __forceinline__ unsigned bf16_rne(float f) {
  const unsigned u = __float_as_uint(f);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ unsigned bf16_pair(double lo, double hi) {
  return bf16_rne((float)lo) | (bf16_rne((float)hi) << 16);
}

// LDS tiles of one stage.
//   fp32: A [k][m] with a row stride of 16 mod 64 floats (the four lane groups
//         of a fragment read, at k .. k + 3, fall in distinct banks); B [n][k']
//         where k sits at position (k mod 4) * 8 + k / 4, so that a lane's eight
//         values of a chunk (its lane group's k of each instruction) are
//         contiguous; rows of 36 floats keep the 16-byte reads of 16 rows on
//         distinct banks.
//   bf16: both [row][k], rows of 40 halves (80 bytes: 16-byte reads of 16 rows
//         on distinct banks).
template <bool F32, int BM, int BN>
struct Tile {
  static constexpr int SA = F32 ? BM + 16 : 20;          // words per row
  static constexpr int SB = F32 ? 36 : 20;
  static constexpr int A_WORDS = F32 ? BK * SA : BM * SA;
  static constexpr int B_WORDS = BN * SB;
  static constexpr int STAGE = A_WORDS + B_WORDS;
};

template <bool F32, int BM, int BN, int NT>
__global__ __launch_bounds__(NT, NT / 128) void k_rounded(
    int M, int N, int K, double alpha, const double* const* __restrict__ Ap, int64_t lda,
    const double* const* __restrict__ Bp, int64_t ldb, double beta, double* const* __restrict__ Cp,
    int64_t ldc, int tiles_m, int tiles_per_inst, int64_t total_tiles, int64_t per_xcd) {
  // the epilogue's binary64 roundings are the ones written
#pragma clang fp contract(off)
  using T = Tile<F32, BM, BN>;
  __shared__ __align__(16) unsigned lds[2 * T::STAGE];
  const int64_t bid = blockIdx.x;
  const int64_t id = (bid % 8) * per_xcd + bid / 8;   // contiguous tiles per XCD
  if (id >= total_tiles) return;
  const int64_t inst = id / tiles_per_inst;
  const int tt = (int)(id - inst * tiles_per_inst);
  const int m0 = (tt % tiles_m) * BM, n0 = (tt / tiles_m) * BN;
  const gcptr A = (gcptr)Ap[inst];
  const gcptr B = (gcptr)Bp[inst];
  const gptr C = (gptr)Cp[inst];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int WM = BM / 2, WN = BN / (NT / 128), FA = WM / 16, FB = WN / 16;
  const int wm0 = (wave & 1) * WM, wn0 = (wave >> 1) * WN;
  const int li = lane & 15, lg = lane >> 4;

  // Load roles.  A: rows m0 + ar, + 1 at k = ka .. ka + PA - 1 (consecutive
  // lanes on consecutive row pairs of a column); B: pairs k = 2 bk, + 1 of
  // columns bc + BR it (sixteen lanes on one column's 256 bytes).
  constexpr int PA = BM * 16 / NT, PB = BN * 16 / NT, BR = NT / 16;
  const int ar = 2 * (tid % (BM / 2)), ka = PA * (tid / (BM / 2));
  const int bk = tid % 16, bc = tid / 16;
  const bool a_full = m0 + BM <= M;
  // Rows and columns outside the matrix re-read the last one: they only
  // reach C entries outside C, which are not stored.
  const gcptr pa0 = A + min(m0 + ar, M - 1), pa1 = A + min(m0 + ar + 1, M - 1);
  d2 av[PA], bv[PB];

  auto load = [&](int k0) {
    if (k0 + BK <= K) {
      if (a_full) {
#pragma unroll
        for (int j = 0; j < PA; ++j)
          av[j] = *(const AS_GLOBAL d2u*)(pa0 + (int64_t)(k0 + ka + j) * lda);
      } else {
#pragma unroll
        for (int j = 0; j < PA; ++j) {
          const int64_t o = (int64_t)(k0 + ka + j) * lda;
          av[j] = d2{pa0[o], pa1[o]};
        }
      }
#pragma unroll
      for (int it = 0; it < PB; ++it)
        bv[it] = *(const AS_GLOBAL d2u*)(B + k0 + 2 * bk +
                                         (int64_t)min(n0 + bc + BR * it, N - 1) * ldb);
    } else {
      // last chunk, partial in k: clamped addresses, zeros beyond K
#pragma unroll
      for (int j = 0; j < PA; ++j) {
        const int k = k0 + ka + j;
        const int64_t o = (int64_t)min(k, K - 1) * lda;
        const double x0 = pa0[o], x1 = pa1[o];
        av[j] = d2{k < K ? x0 : 0.0, k < K ? x1 : 0.0};
      }
      const int k = k0 + 2 * bk;
#pragma unroll
      for (int it = 0; it < PB; ++it) {
        const gcptr p = B + (int64_t)min(n0 + bc + BR * it, N - 1) * ldb;
        const double x0 = p[min(k, K - 1)], x1 = p[min(k + 1, K - 1)];
        bv[it] = d2{k < K ? x0 : 0.0, k + 1 < K ? x1 : 0.0};
      }
    }
  };
  auto store = [&](int stage) {
    unsigned* sa = lds + stage * T::STAGE;
    unsigned* sb = sa + T::A_WORDS;
    if constexpr (F32) {
#pragma unroll
      for (int j = 0; j < PA; ++j)
        *(f2*)(sa + (ka + j) * T::SA + ar) = f2{(float)av[j].x, (float)av[j].y};
      const int pos = ((2 * bk) & 3) * 8 + (bk >> 1);
#pragma unroll
      for (int it = 0; it < PB; ++it) {
        unsigned* row = sb + (bc + BR * it) * T::SB + pos;
        row[0] = __float_as_uint((float)bv[it].x);
        row[8] = __float_as_uint((float)bv[it].y);
      }
    } else {
      unsigned w0[PA / 2], w1[PA / 2];
#pragma unroll
      for (int j = 0; j < PA / 2; ++j) {
        w0[j] = bf16_pair(av[2 * j].x, av[2 * j + 1].x);
        w1[j] = bf16_pair(av[2 * j].y, av[2 * j + 1].y);
      }
      unsigned* r0 = sa + ar * T::SA + ka / 2;
#pragma unroll
      for (int j = 0; j < PA / 2; ++j) {
        r0[j] = w0[j];
        r0[T::SA + j] = w1[j];
      }
#pragma unroll
      for (int it = 0; it < PB; ++it)
        sb[(bc + BR * it) * T::SB + bk] = bf16_pair(bv[it].x, bv[it].y);
    }
  };

  f4 acc[FA][FB];
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

  const int nk = (K + BK - 1) / BK;
  load(0);
  store(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) load((kt + 1) * BK);
    const unsigned* sa = lds + (kt & 1) * T::STAGE;
    const unsigned* sb = sa + T::A_WORDS;
    if constexpr (F32) {
      f4 fb[FB][2];
#pragma unroll
      for (int j = 0; j < FB; ++j)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          fb[j][u] = *(const f4*)(sb + (wn0 + 16 * j + li) * T::SB + 8 * lg + 4 * u);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float fa[FA];
#pragma unroll
        for (int i = 0; i < FA; ++i)
          fa[i] = __uint_as_float(sa[(4 * t + lg) * T::SA + wm0 + 16 * i + li]);
#pragma unroll
        for (int i = 0; i < FA; ++i)
#pragma unroll
          for (int j = 0; j < FB; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][t >> 2][t & 3], fa[i],
                                                             acc[i][j], 0, 0, 0);
      }
    } else {
      bf8 fa[FA], fb[FB];
#pragma unroll
      for (int i = 0; i < FA; ++i)
        fa[i] = __builtin_bit_cast(bf8, *(const u4*)(sa + (wm0 + 16 * i + li) * T::SA + 4 * lg));
#pragma unroll
      for (int j = 0; j < FB; ++j)
        fb[j] = __builtin_bit_cast(bf8, *(const u4*)(sb + (wn0 + 16 * j + li) * T::SB + 4 * lg));
#pragma unroll
      for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) store((kt + 1) & 1);
    __syncthreads();
  }

  // epilogue: lane holds C(m0 + wm0 + 16 i + li, n0 + wn0 + 16 j + 4 lg + v).
  // Nontemporal only where the columns are whole 128-byte lines: two tiles, or
  // two columns, may share a line otherwise, and its parts reach memory one by
  // one (432 x 450 x 91 x 11 in binary32: 93 us so, 42 us with ordinary stores).
  const auto write = [&](auto lines) {
#pragma unroll
    for (int i = 0; i < FA; ++i) {
      const int row = m0 + wm0 + 16 * i + li;
      double cv[FB][4];
      if (beta != 0.0) {
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int col = n0 + wn0 + 16 * j + 4 * lg + v;
            cv[j][v] = C[min(row, M - 1) + (int64_t)min(col, N - 1) * ldc];
          }
      }
#pragma unroll
      for (int j = 0; j < FB; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int col = n0 + wn0 + 16 * j + 4 * lg + v;
          double x = alpha * (double)acc[i][j][v];
          if (beta != 0.0) x = x + beta * cv[j][v];
          const gptr p = C + row + (int64_t)col * ldc;
          if (row < M && col < N) {
            if constexpr (lines) __builtin_nontemporal_store(x, p);
            else *p = x;
          }
        }
    }
  };
  if ((((uintptr_t)C | (uintptr_t)(8 * ldc)) & 127) == 0) write(std::true_type{});
  else write(std::false_type{});
}

template <bool F32, int BM, int BN, int NT>
static hipError_t launch(const UniformArgs& a, hipStream_t s) {
  const int tiles_m = (a.m + BM - 1) / BM, tiles_n = (a.n + BN - 1) / BN;
  const int64_t tpi = (int64_t)tiles_m * tiles_n;
  return launch_in_parts(tpi, a.batch, NT, [&](int64_t b0, int64_t total, int64_t per_xcd,
                                               dim3 grid) {
    hipLaunchKernelGGL((k_rounded<F32, BM, BN, NT>), grid, dim3(NT), 0, s, a.m, a.n, a.k, a.alpha,
                       a.A + b0, a.lda, a.B + b0, a.ldb, a.beta, a.C + b0, a.ldc, tiles_m, (int)tpi,
                       total, per_xcd);
    return hipGetLastError();
  });
}

// 128 x 128 where neither side is padded further by it than by 64, else 64 x
// 64; a batch too short to give every CU two 128 x 128 tiles also takes the
// smaller one.  Measured, 128 x 128 against 64 x 64 in binary32: 20,000 x
// 256^3 7.75 / 8.92 ms, 20,000 x 96^3 0.89 / 1.01, 300 x 256^3 0.126 / 0.138;
// but 5,000 x 192^3 1.42 / 1.04, 40,000 x 64^3 1.20 / 0.69, 3,000 x 129 x 513 x
// 257 2.97 / 2.46 and, too short, 64 x 256^3 0.031 / 0.028.  128 x 64 and 64 x
// 128 lost to one of the two in binary32 at every size tried.  The 128 x 128
// binary32 tile runs eight waves (7.75 ms against 8.00 with four: its
// products are long enough to hide the conversions of more waves), the
// bfloat16 one four (5.55 against 5.65 ms).
static bool whole128(int x) { return (x + 127) / 128 * 2 == (x + 63) / 64; }

template <bool F32>
static hipError_t pick(const UniformArgs& a, hipStream_t s) {
  const int64_t tiles = (int64_t)((a.m + 127) / 128) * ((a.n + 127) / 128) * a.batch;
  if (whole128(a.m) && whole128(a.n) && tiles >= 2 * (int64_t)a.num_cus)
    return launch<F32, 128, 128, F32 ? 512 : 256>(a, s);
  return launch<F32, 64, 64, 256>(a, s);
}

}  // namespace rounded

hipError_t launch_rounded(const UniformArgs& a, int mode, hipStream_t s) {
  return mode == 1 ? rounded::pick<true>(a, s) : rounded::pick<false>(a, s);
}

}  // namespace bg
