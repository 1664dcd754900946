// Emulated binary64 batched GEMM on the int8 matrix cores of gfx950
// (v_mfma_i32_16x16x64_i8), the i8emu<S> mode.
//
// Same operation as the FP64 path (the paper, Section II, Eq. 1), on binary64
// inputs and outputs.  The error-free splitting follows Ozaki, Ogita, Oishi
// and Rump (Numer. Algorithms 59, 2012), with integer digits:
//   1. e_i: frexp exponent of the largest |A(i, p)| over the whole row i of A;
//      f_j likewise for column j of B (kernel k_exp, one pass over A and B).
//   2. X = rint(A(i, p) 2^(8S-2-e_i)), an integer with |X| <= 2^(8S-2);
//      Y likewise for B.
//   3. Signed base-256 digits X = sum_t d_t 256^(S-t), d_t in [-128, 127]
//      (d_1 in [-64, 64]): with Z = X + 0x80..80 (S bytes), digit d_t is byte
//      S-t of Z minus 128, i.e. that byte with its top bit flipped, read as
//      an int8.
//   4. For each diagonal g = t + u <= S + 1, S_g = sum_p sum_{t+u=g}
//      dA_t(i, p) dB_u(p, j) on the int8 matrix cores in int32: exact, since
//      |S_g| <= S k 2^14 < 2^31 for k <= 8192.  Exact integers do not depend on
//      the order of the sum, so any blocking of k gives the same S_g.
//   5. In binary64: T = S_{S+1}; T = S_g + T 2^-8 for g = S .. 2;
//      V = T 2^(e_i + f_j - 12); C = alpha V (+ beta C).
// Every rounding is fixed in kind and order, so the result equals a CPU
// implementation of these steps bit for bit.
//
// Main kernel: 128 x 64 C tiles, each by a workgroup of eight waves (32 x 32
// apiece, 2 x 2 blocks of 16 x 16), 64 of k per step.  Each thread loads 16
// binary64 values of A (one row, 16 consecutive k) and 8 of B (one column, 8
// consecutive k), turns them into S digit bytes each and writes one word per
// digit plane to LDS; then each wave runs S (S + 1) / 2 x 4 int8 matrix-core
// instructions into S int32 accumulator sets.  The instruction's first operand
// is B's digits and its second A's, so a result block is the transpose of a C
// block and its 16 lanes cover 16 consecutive rows of a C column (coalesced
// epilogue).  NN operands only.
//
// What bounds it: the phases of the one workgroup that a CU holds (the digit
// planes and the accumulators fill LDS and registers), one after another.  At
// 256^3 and S = 7 a tile takes 4 x 3,600 cycles of matrix cores per SIMD and
// about as many of vector instructions for the split, where memory alone takes
// 5.7 of the kernel's 12.7 ms per 20,000 instances.  So a workgroup takes tile
// after tile, and the values of the next step, or of the next tile's first, are
// in flight during a step's products and the epilogue; the split rounds by one
// fused multiply-add per value (six operations beyond six digits), where a
// scaling, rint and integer conversion took three times as many; digits lie in
// LDS without bank conflicts.  Measured with the exponent pass (3.5 ms), 20,000
// x 256^3: S = 5 16.8 -> 13.8 ms, S = 7 18.2 -> 16.3, S = 8 19.4 -> 18.0; beta
// 1, 5,000 instances, S = 5: 6.2 -> 4.0 ms.  Four waves per SIMD on 64 x 64
// tiles do not fit the registers (S = 7 spills: 26 ms).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bgemm_internal.h"

namespace bg {
namespace emu8 {

typedef int i4 __attribute__((ext_vector_type(4)));
#define AS_GLOBAL __attribute__((address_space(1)))
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef double d2 __attribute__((ext_vector_type(2)));

// C tile: TM x BN by NT threads, BK of k per step
constexpr int TM = 128, BN = 64, BK = 64, NT = 512;
constexpr int PLANE_A = TM * BK;       // bytes per digit plane of A
constexpr int PLANE_B = BN * BK;       // bytes per digit plane of B

// Where the 16 digits k = 16 c .. 16 c + 15 of row r lie in a plane.  A 16-byte
// LDS read serves lanes {0-3, 12-15, 20-27} of a wave's first half together, then
// the others: with these offsets such a group's rows meet all 64 banks once.
__device__ __forceinline__ int slot(int r, int c) {
  return r * BK + 16 * ((c ^ -(r >> 2)) & 3);
}

constexpr int EXP_COLS = 16;           // columns of B per exponent block

// ---- exponents ------------------------------------------------------------

__device__ __forceinline__ int frexp_exp(double mx) {
  int e = 0;
  (void)frexp(mx, &e);
  return mx > 0.0 ? e : 0;
}

// Blocks [0, nb_a) of an instance: one row of A per thread; blocks
// [nb_a, nb_a + nb_b): EXP_COLS columns of B, one wave per column at a time.
__global__ __launch_bounds__(256) void k_exp(int M, int N, int K,
                                             const double* const* __restrict__ Ap, int64_t lda,
                                             const double* const* __restrict__ Bp, int64_t ldb,
                                             int* __restrict__ ea, int* __restrict__ fb, int nb_a,
                                             int per_inst) {
  const int64_t inst = blockIdx.x / per_inst;
  const int blk = (int)(blockIdx.x - inst * per_inst);
  if (blk < nb_a) {
    const int r = blk * 256 + threadIdx.x;
    if (r >= M) return;
    const double* A = Ap[inst] + r;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0, m3 = 0.0;
    int p = 0;
    for (; p + 4 <= K; p += 4) {
      m0 = fmax(m0, fabs(A[(int64_t)p * lda]));
      m1 = fmax(m1, fabs(A[(int64_t)(p + 1) * lda]));
      m2 = fmax(m2, fabs(A[(int64_t)(p + 2) * lda]));
      m3 = fmax(m3, fabs(A[(int64_t)(p + 3) * lda]));
    }
    for (; p < K; ++p) m0 = fmax(m0, fabs(A[(int64_t)p * lda]));
    ea[inst * M + r] = frexp_exp(fmax(fmax(m0, m1), fmax(m2, m3)));
  } else {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = (blk - nb_a) * EXP_COLS;
    for (int c = c0 + wave; c < c0 + EXP_COLS && c < N; c += 4) {
      const double* B = Bp[inst] + (int64_t)c * ldb;
      double mx = 0.0;
      for (int p = lane; p < K; p += 64) mx = fmax(mx, fabs(B[p]));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
      if (lane == 0) fb[inst * N + c] = frexp_exp(mx);
    }
  }
}

// ---- digits ---------------------------------------------------------------

// Scales of a row or column whose values are to be multiplied by 2^sh: a shift
// beyond what one factor holds (rows of values below 2^-960) is split in two.
struct Scale {
  double pre;    // 1, or 2^512 on such rows
  double f;      // 2^sh / pre
  double fh;     // f 2^-32
};
__device__ __forceinline__ Scale make_scale(int sh) {
  const bool far = sh > 1000;
  const double f = ldexp(1.0, far ? sh - 512 : sh);
  return Scale{far ? 0x1p512 : 1.0, f, f * 0x1p-32};
}

// Z = X + 0x80..80 (S bytes) for X = rint(v 2^sh): low and high words (bytes
// beyond S are not meaningful).  Adding 1.5 2^52 rounds to an integer, ties to
// even, and leaves it in the sum's low bits, the digits' offset with it, so up
// to six digits take one fused multiply-add.  Beyond, X is split at 2^32: h =
// rint(v 2^(sh-32)), l = v 2^sh - h 2^32 exactly, and rint(X) = h 2^32 + rint(l);
// l + 0x80808080 is positive and may carry into the high word.
template <int S>
__device__ __forceinline__ void z_words(double v, const Scale& sc, unsigned& lo, unsigned& hi) {
  constexpr unsigned ML = S >= 4 ? 0x80808080u : (unsigned)(0x80808080ull >> (8 * (4 - S)));
  constexpr unsigned MH = S > 4 ? (unsigned)(0x80808080ull >> (8 * (8 - S))) : 0u;
  constexpr double BIG = 0x1.8p52;
  if constexpr (S <= 6) {
    const double t = __builtin_fma(v, sc.f, BIG + ((double)MH * 0x1p32 + (double)ML));
    const uint64_t b = __builtin_bit_cast(uint64_t, t);
    lo = (unsigned)b;
    hi = (unsigned)(b >> 32);
  } else {
    const double x = v * sc.f;
    const double th = __builtin_fma(v, sc.fh, BIG + (double)MH);
    const double l = __builtin_fma(th - (BIG + (double)MH), -0x1p32, x);
    const double tl = l + (BIG + (double)ML);
    const uint64_t bh = __builtin_bit_cast(uint64_t, th), bl = __builtin_bit_cast(uint64_t, tl);
    lo = (unsigned)bl;
    hi = (unsigned)bh + (unsigned)(bl >> 32) - 0x43380000u;
  }
}

// 4 x 4 byte transpose: out[b] = [w0.b, w1.b, w2.b, w3.b] (first word in the
// low byte), for the NB lowest bytes b.  v_perm_b32 picks bytes of
// {src0 (high), src1 (low)}: selectors 0-3 address src1, 4-7 src0.
template <int NB>
__device__ __forceinline__ void transpose4(unsigned w0, unsigned w1, unsigned w2, unsigned w3,
                                           unsigned (&out)[4]) {
  const unsigned l01 = __builtin_amdgcn_perm(w1, w0, 0x05010400u);   // w0.0 w1.0 w0.1 w1.1
  const unsigned l23 = __builtin_amdgcn_perm(w3, w2, 0x05010400u);   // w2.0 w3.0 w2.1 w3.1
  out[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u);
  if constexpr (NB > 1) out[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u);
  if constexpr (NB > 2) {
    const unsigned h01 = __builtin_amdgcn_perm(w1, w0, 0x07030602u); // w0.2 w1.2 w0.3 w1.3
    const unsigned h23 = __builtin_amdgcn_perm(w3, w2, 0x07030602u);
    out[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u);
    if constexpr (NB > 3) out[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
  }
}

// NV values (consecutive k, NV = 8 or 16) -> S digit planes, one NV-byte word
// each, at dst + t * plane (t = 0 the most significant digit).
template <int S, int NV>
__device__ __forceinline__ void split(const double* v, const Scale& sc, unsigned char* dst,
                                      int plane) {
  constexpr int NL = S < 4 ? S : 4, NH = S - NL, NQ = NV / 4;
  unsigned w[S][NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    unsigned lo[4], hi[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) z_words<S>(v[4 * q + j], sc, lo[j], hi[j]);
    unsigned bl[4], bh[4];
    transpose4<NL>(lo[0], lo[1], lo[2], lo[3], bl);
#pragma unroll
    for (int b = 0; b < NL; ++b) w[S - 1 - b][q] = bl[b] ^ 0x80808080u;
    if constexpr (NH > 0) {
      transpose4<NH>(hi[0], hi[1], hi[2], hi[3], bh);
#pragma unroll
      for (int b = 0; b < NH; ++b) w[S - 5 - b][q] = bh[b] ^ 0x80808080u;
    }
  }
#pragma unroll
  for (int t = 0; t < S; ++t) {
    if constexpr (NQ == 4) *(u4*)(dst + t * plane) = u4{w[t][0], w[t][1], w[t][2], w[t][3]};
    else *(u2*)(dst + t * plane) = u2{w[t][0], w[t][1]};
  }
}

// ---- main kernel ----------------------------------------------------------

// x if ok, else +0.0, by masking its bits: the value is used either way, so
// the compiler keeps the load unconditional (no branch and wait per load)
__device__ __forceinline__ double keep(double x, bool ok) {
  const uint64_t m = ok ? ~0ull : 0ull;
  return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, x) & m);
}

template <int S>
__global__ __launch_bounds__(NT, 2) void k_emu8(int M, int N, int K, double alpha,
                                                const double* const* __restrict__ Ap, int64_t lda,
                                                const double* const* __restrict__ Bp, int64_t ldb,
                                                double beta, double* const* __restrict__ Cp,
                                                int64_t ldc, const int* __restrict__ ea,
                                                const int* __restrict__ fb, int tiles_m,
                                                int tiles_per_inst, int64_t total_tiles,
                                                int64_t per_xcd) {
  // every binary64 rounding below is the one written (no fused multiply-add)
#pragma clang fp contract(off)
  // Eight digits leave no registers for the next step's values, nor for what a
  // loop over tiles keeps (either spills: 29 and 20.4 ms against 18.6).
  constexpr bool AHEAD = S < 8;
  // A's leading digit planes stay in registers over B's, the others are read
  // again for each (they meet few of B's); one to eight measured the same.
  constexpr int HELD = S < 3 ? S : 3;
  __shared__ __align__(16) unsigned char lds[S * (PLANE_A + PLANE_B)];
  __shared__ int se[2][TM + BN];       // exponents of a tile's rows and columns
  unsigned char* la = lds;
  unsigned char* lb = lds + S * PLANE_A;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // split roles: A row m0 + ar, k = 16 akg .. +15; B column n0 + bc, k = 8 bkg .. +7
  const int ar = tid % TM, akg = tid / TM;
  const int bc = tid >> 3, bkg = tid & 7;
  // wave tile: rows wm0 .. +31, columns wn0 .. +31 of the C tile
  const int wm0 = (wave & 3) * 32, wn0 = (wave >> 2) * 32;
  const int li = lane & 15, lg = lane >> 4;
  unsigned char* const wa = la + slot(ar, akg);
  unsigned char* const wb = lb + slot(bc, bkg >> 1) + 8 * (bkg & 1);
  const unsigned char* const ra = la + slot(wm0 + li, lg);
  const unsigned char* const rb = lb + slot(wn0 + li, lg);

  // Tiles of this workgroup: ids first, first + stride, ... of its XCD's share
  const int64_t first = (blockIdx.x % 8) * per_xcd;
  const int64_t end = min(first + per_xcd, total_tiles);
  const int64_t stride = gridDim.x / 8;
  int64_t id = first + blockIdx.x / 8;
  if (id >= end) return;

  double av[16], bv[8];
  int ax, bx;                          // exponents of this thread's row and column
  const AS_GLOBAL double* arow;
  const AS_GLOBAL double* bcol;
  bool b_vec;
  auto place = [&](int64_t t) {
    const int64_t inst = t / tiles_per_inst;
    const int tt = (int)(t - inst * tiles_per_inst);
    const int m0 = (tt % tiles_m) * TM, n0 = (tt / tiles_m) * BN;
    const double* B = Bp[inst];
    b_vec = ((((uintptr_t)B) & 15) == 0) && ((ldb & 1) == 0);
    // out-of-range rows / columns read row / column 0 of the matrix (their sums
    // are never stored)
    const int r = m0 + ar < M ? m0 + ar : 0, c = n0 + bc < N ? n0 + bc : 0;
    arow = (const AS_GLOBAL double*)Ap[inst] + r;
    bcol = (const AS_GLOBAL double*)B + (int64_t)c * ldb;
    ax = ea[inst * M + r];
    bx = fb[inst * N + c];
  };
  // every load of a step is issued before the first wait
  auto load = [&](int k0) {
    const int ka = k0 + 16 * akg, kb = k0 + 8 * bkg;
    if (k0 + BK <= K) {
      // whole step inside k (uniform): plain loads
      const AS_GLOBAL double* pa = arow + (int64_t)ka * lda;
#pragma unroll
      for (int j = 0; j < 16; ++j) av[j] = pa[(int64_t)j * lda];
      if (b_vec) {
        const AS_GLOBAL d2* p = (const AS_GLOBAL d2*)(bcol + kb);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const d2 x = p[j];
          bv[2 * j] = x.x;
          bv[2 * j + 1] = x.y;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) bv[j] = bcol[kb + j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) av[j] = arow[(int64_t)min(ka + j, K - 1) * lda];
#pragma unroll
      for (int j = 0; j < 8; ++j) bv[j] = bcol[min(kb + j, K - 1)];
    }
  };

  place(id);
  if constexpr (AHEAD) load(0);
  for (int par = 0;; par ^= 1) {
    // the epilogue reads the exponents here, not at the latency of memory; the
    // tile before it may still be reading the other half
    if (akg == 0) se[par][ar] = ax;
    if (bkg == 0) se[par][TM + bc] = bx;
    const Scale asc = make_scale((8 * S - 2) - ax), bsc = make_scale((8 * S - 2) - bx);
    const bool far = __any(asc.pre != 1.0 || bsc.pre != 1.0);
    const int64_t next = id + stride;

    i4 acc[S][2][2];
#pragma unroll
    for (int g = 0; g < S; ++g)
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) acc[g][bi][bj] = i4{0, 0, 0, 0};

    for (int k0 = 0; k0 < K; k0 += BK) {
      if constexpr (!AHEAD) load(k0);
      if (k0 + BK > K) {
#pragma unroll
        for (int j = 0; j < 16; ++j) av[j] = keep(av[j], k0 + 16 * akg + j < K);
#pragma unroll
        for (int j = 0; j < 8; ++j) bv[j] = keep(bv[j], k0 + 8 * bkg + j < K);
      }
      if (far) {
#pragma unroll
        for (int j = 0; j < 16; ++j) av[j] *= asc.pre;
#pragma unroll
        for (int j = 0; j < 8; ++j) bv[j] *= bsc.pre;
      }
      __syncthreads();   // the previous step's digit reads are done
      split<S, 16>(av, asc, wa, PLANE_A);
      split<S, 8>(bv, bsc, wb, PLANE_B);
      if constexpr (AHEAD) {
        // the next values are in flight through the products below
        asm volatile("" ::: "memory");
        int kn = k0 + BK;
        if (kn >= K && next < end) {
          place(next);
          kn = 0;
        }
        if (kn < K) load(kn);
        asm volatile("" ::: "memory");
      }
      __syncthreads();

      auto read_a = [&](int t, i4 (&f)[2]) {
#pragma unroll
        for (int bi = 0; bi < 2; ++bi) f[bi] = *(const i4*)(ra + t * PLANE_A + 16 * bi * BK);
      };
      i4 af[HELD][2];
#pragma unroll
      for (int t = 0; t < HELD; ++t) read_a(t, af[t]);
#pragma unroll
      for (int u = 0; u < S; ++u) {
        i4 bf[2];
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) bf[bj] = *(const i4*)(rb + u * PLANE_B + 16 * bj * BK);
#pragma unroll
        for (int t = 0; t + u < S; ++t) {
          i4 at[2];
          if (t < HELD) {
            at[0] = af[t < HELD ? t : 0][0];
            at[1] = af[t < HELD ? t : 0][1];
          } else {
            read_a(t, at);
          }
#pragma unroll
          for (int bi = 0; bi < 2; ++bi)
#pragma unroll
            for (int bj = 0; bj < 2; ++bj)
              acc[t + u][bi][bj] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                  bf[bj], at[bi], acc[t + u][bi][bj], 0, 0, 0);
        }
      }
    }

    // epilogue: lane (li, lg), register v of block (bi, bj) holds the diagonal
    // sums of C(row m0 + wm0 + 16 bi + li, column n0 + wn0 + 16 bj + 4 lg + v)
    const int64_t inst = id / tiles_per_inst;
    const int tt = (int)(id - inst * tiles_per_inst);
    const int m0 = (tt % tiles_m) * TM, n0 = (tt / tiles_m) * BN;
    AS_GLOBAL double* C = (AS_GLOBAL double*)Cp[inst];
    // this lane's place, computed here: kept from tile to tile, the offsets that
    // follow from it would take the registers of the loads in flight
    int el = threadIdx.x;
    asm volatile("" : "+v"(el));
    const int r0 = ((el >> 6) & 3) * 32 + (el & 15);
    const int c0 = (el >> 8) * 32 + 4 * ((el >> 4) & 3);
    // Four of C's values are read together before they are used: 5,000 x 256^3
    // with five digits and beta 1: 4.65 ms one by one, 3.93 so.
    auto write = [&](auto add, auto lines) {
#pragma unroll
      for (int bi = 0; bi < 2; ++bi) {
        const int r = r0 + 16 * bi;
        if (m0 + r >= M) continue;
        const int er = se[par][r];
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
          const int c = c0 + 16 * bj;
          AS_GLOBAL double* cp = C + (m0 + r) + (int64_t)(n0 + c) * ldc;
          [[maybe_unused]] double cv[4];
          if constexpr (add)
#pragma unroll
            for (int v = 0; v < 4; ++v)
              cv[v] = cp[(int64_t)min(v, N - 1 - n0 - c) * ldc];   // a column inside
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (n0 + c + v >= N) continue;
            double T = (double)acc[S - 1][bi][bj][v];
#pragma unroll
            for (int g = S - 2; g >= 0; --g) T = (double)acc[g][bi][bj][v] + T * 0x1p-8;
            const double V = ldexp(T, er + se[par][TM + c + v] - 12);
            double x = alpha * V;
            if constexpr (add) x = x + beta * cv[v];
            if constexpr (lines) __builtin_nontemporal_store(x, cp + (int64_t)v * ldc);
            else cp[(int64_t)v * ldc] = x;
          }
        }
      }
    };
    // nontemporal where the columns are whole 128-byte lines, as no other tile
    // writes to these (5,000 x 256^3, five digits: 3.54 -> 3.48 ms)
    if (beta != 0.0) write(std::true_type{}, std::false_type{});
    else if ((((uintptr_t)C | (uintptr_t)(8 * ldc)) & 127) == 0)
      write(std::false_type{}, std::true_type{});
    else write(std::false_type{}, std::false_type{});
    if constexpr (!AHEAD) return;
    id = next;
    if (id >= end) return;
  }
}

template <int S>
static hipError_t launch_group(const UniformArgs& a, int64_t b0, int g, int* ea, int* fb,
                               hipStream_t s) {
  const int nb_a = (a.m + 255) / 256, nb_b = (a.n + EXP_COLS - 1) / EXP_COLS;
  const int per_inst = nb_a + nb_b;
  hipLaunchKernelGGL(k_exp, dim3((unsigned)((int64_t)per_inst * g)), dim3(256), 0, s, a.m, a.n,
                     a.k, a.A + b0, a.lda, a.B + b0, a.ldb, ea, fb, nb_a, per_inst);
  const int tiles_m = (a.m + TM - 1) / TM, tiles_n = (a.n + BN - 1) / BN;
  const int64_t tpi = (int64_t)tiles_m * tiles_n;
  const int64_t total = tpi * g;
  const int64_t per_xcd = (total + 7) / 8;
  // A grid of two workgroups per CU takes all tiles between them, each XCD's its
  // contiguous share (from two digits on registers hold one of the two at a time,
  // 137 to 256 a lane); with eight digits one workgroup takes one tile.
  const int64_t per = S == 8 ? per_xcd : std::min<int64_t>(per_xcd, std::max(1, a.num_cus / 4));
  hipLaunchKernelGGL((k_emu8<S>), dim3((unsigned)(per * 8)), dim3(NT), 0, s, a.m, a.n, a.k,
                     a.alpha, a.A + b0, a.lda, a.B + b0, a.ldb, a.beta, a.C + b0, a.ldc, ea, fb,
                     tiles_m, (int)tpi, total, per_xcd);
  return hipGetLastError();
}

template <int S>
static hipError_t launch(const UniformArgs& a, void* ws, size_t ws_bytes, hipStream_t s) {
  const int64_t per = (int64_t)(a.m + a.n) * (int64_t)sizeof(int);
  int64_t gmax = (int64_t)(ws_bytes / (size_t)per);
  const int tiles_m = (a.m + TM - 1) / TM, tiles_n = (a.n + BN - 1) / BN;
  const int64_t tpi = (int64_t)tiles_m * tiles_n;
  const int nb = (a.m + 255) / 256 + (a.n + EXP_COLS - 1) / EXP_COLS;
  // both launches of a group stay within the launch limit (the tile loop's grid
  // does not grow with the group)
  gmax = std::min<int64_t>(gmax, instances_per_launch(nb, 256));
  gmax = std::min<int64_t>(gmax, S == 8 ? instances_per_launch(tpi, NT) : (INT32_MAX - 8) / tpi);
  if (gmax < 1) return hipErrorInvalidValue;
  for (int64_t b0 = 0; b0 < a.batch; b0 += gmax) {
    const int g = (int)std::min<int64_t>(gmax, a.batch - b0);
    int* ea = (int*)ws;
    int* fb = ea + (int64_t)g * a.m;
    const hipError_t e = launch_group<S>(a, b0, g, ea, fb, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace emu8

hipError_t launch_emu8(const UniformArgs& a, int slices, void* ws, size_t ws_bytes,
                       hipStream_t s) {
  using namespace emu8;
  switch (slices) {
    case 1: return launch<1>(a, ws, ws_bytes, s);
    case 2: return launch<2>(a, ws, ws_bytes, s);
    case 3: return launch<3>(a, ws, ws_bytes, s);
    case 4: return launch<4>(a, ws, ws_bytes, s);
    case 5: return launch<5>(a, ws, ws_bytes, s);
    case 6: return launch<6>(a, ws, ws_bytes, s);
    case 7: return launch<7>(a, ws, ws_bytes, s);
    case 8: return launch<8>(a, ws, ws_bytes, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace bg
