// Internal declarations shared by the C-ABI layer (bgemm_api.cpp) and the
// kernel launchers (bgemm_kernels.hip).  Not part of the public interface.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/bgemm.h"

namespace bg {

// Tile shapes: one configuration of a tile kernel, C tile BM x BN per workgroup
// on the 4x4x4 FP64 matrix-core form.
enum TileClass : int {
  TC_32 = 0,      // 32 x 32 tile
  TC_64 = 1,      // 64 x 64 tile
  TC_128 = 2,     // 128 x 128 tile
  TC_COUNT = 3,   // classes a caller can force
  TC_128x64 = 3,
  TC_64x32 = 4,
  TC_32x64 = 5,
  TC_32x16 = 6,
  TC_128x48 = 7,
  TC_SHAPES = 8
};

// Picks the tile class for a uniform batch of `batch` instances (`nn`: neither
// operand transposed) on a device of `num_cus` compute units; `force` >= 0
// overrides.
TileClass pick_uniform_class(bool nn, int m, int n, int k, int batch, int num_cus, int force);

// For tests and timing, exported beside the public interface: the shape that a
// uniform batch takes by default, and a handle's override by any of the shapes
// (-1 none; bg_set_uniform_class knows the first three).
extern "C" int bgi_pick_tile(int nn, int m, int n, int k, int batch, int num_cus);
extern "C" bg_status_t bgi_force_tile(bg_handle_t h, int shape);

// Instances one launch may take at `blocks` workgroups of `threads` each (0: not
// even one).  A launch counts its threads in 32 bits and drops the rest without
// an error; workgroups are dealt to the XCDs in whole turns of eight.
inline int64_t instances_per_launch(int64_t blocks, int threads) {
  const int64_t most = (((int64_t)1 << 32) - 1) / threads / 8 * 8;
  return most / blocks;
}

// Launches a uniform batch whose instances take `tiles` workgroups of `threads`
// each, in as few parts as the launch limit allows: part(first instance, tiles of
// the part, tiles per XCD, workgroups).  hipErrorInvalidValue for grids beyond
// int32 over the whole batch.
template <class Part>
hipError_t launch_in_parts(int64_t tiles, int batch, int threads, Part part) {
  if (tiles > INT32_MAX || (tiles * batch + 7) / 8 * 8 > INT32_MAX) return hipErrorInvalidValue;
  const int64_t per = instances_per_launch(tiles, threads);
  if (per < 1) return hipErrorInvalidValue;
  for (int64_t first = 0; first < batch; first += per) {
    const int64_t total = tiles * (batch - first < per ? batch - first : per);
    const int64_t per_xcd = (total + 7) / 8;
    const hipError_t e = part(first, total, per_xcd, dim3((unsigned)(per_xcd * 8)));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

struct UniformArgs {
  bool ta, tb;
  int m, n, k;
  double alpha, beta;
  const double* const* A; int64_t lda;
  const double* const* B; int64_t ldb;
  double* const* C; int64_t ldc;
  int batch;
  int num_cus = 0;   // compute units of the device
};

// Launches the uniform batched GEMM (product path; alpha != 0, k > 0).
hipError_t launch_uniform(const UniformArgs& a, TileClass cls, hipStream_t s);

// Batches of n x n products C_i <- A_i B_i (ld = n), one per size: short batches
// share launches, in the given order; a batch that fills the chip runs alone.
struct SquareGroup {
  int n, batch;
  const double* const* A;
  const double* const* B;
  double* const* C;
};
hipError_t launch_square_groups(const SquareGroup* groups, int count, int num_cus, hipStream_t s);
// The same on a handle's device and stream (one call per size when the caller
// has forced a tile class on the handle).
bg_status_t dgemm_square_groups(bg_handle_t h, const SquareGroup* groups, int count);

// Reduced precision modes of the uniform batch (NN operands only): mode 1
// binary32, 2 bfloat16.  hipErrorInvalidValue for grids beyond int32.
hipError_t launch_rounded(const UniformArgs& a, int mode, hipStream_t s);
// Emulated precision modes (NN operands only): mode 3 emulated binary64 with
// `slices` (1..8) bfloat16 digit slices, 5 the same digits summed in binary32.
// hipErrorInvalidValue for grids beyond int32.
hipError_t launch_uniform_lowp(const UniformArgs& a, int mode, int slices, hipStream_t s);
// Emulated binary64 on int8 digit slices (NN, k <= 8192): per group of
// instances, row / column exponents into the workspace (m + n ints per
// instance), then the product.  hipErrorInvalidValue when the workspace holds
// no instance or slices is outside 1..8.
hipError_t launch_emu8(const UniformArgs& a, int slices, void* ws, size_t ws_bytes, hipStream_t s);

// Launches C_i <- beta * C_i (beta != 1) for every instance, used when the
// product term vanishes (alpha == 0 or k == 0).
hipError_t launch_scale(double beta, double* const* C, int64_t ldc, int m, int n, int batch,
                        hipStream_t s);

struct VbatchedArgs {
  bool ta, tb;
  const int *m, *n, *k;
  double alpha, beta;
  const double* const* A; const int* lda;
  const double* const* B; const int* ldb;
  double* const* C; const int* ldc;
  int batch;
  int* info;  // nullable
};

// Host-side argument rules of the variable-size call (0 when valid, else the
// reference-BLAS argument number) and the argument pack built from them.
int vbatched_host_args(char transa, char transb, const int* d_m, const int* d_n, const int* d_k,
                       const void* dA, const int* d_lda, const void* dB, const int* d_ldb,
                       const void* dC, const int* d_ldc, int batch);
VbatchedArgs vbatched_args(char transa, char transb, const int* d_m, const int* d_n,
                           const int* d_k, double alpha, const double* const* dA,
                           const int* d_lda, const double* const* dB, const int* d_ldb,
                           double beta, double* const* dC, const int* d_ldc, int batch,
                           int* d_info);

// Workspace layout used by the vbatched planner and executor.
struct VbWorkspace {
  void* base;
  size_t bytes;
};

// Bytes of workspace the planner needs for `batch` instances, excluding the
// optional tile map (which uses whatever remains).
size_t vbatched_workspace_bytes(int batch);

// Plans (validate, count tiles, prefix sums, tile map) and executes the
// variable-size batch with a persistent kernel; all on stream `s`.
hipError_t launch_vbatched(const VbatchedArgs& a, const VbWorkspace& ws, int num_cus,
                           hipStream_t s);

// Complex uniform batch (interleaved binary64 pairs; ld in complex elements;
// op codes 0 N, 1 T, 2 C; alpha and beta point to host (re, im) pairs).
struct ZUniformArgs {
  int ta, tb;
  int m, n, k;
  const double* alpha;
  const double* beta;
  const double* const* A; int64_t lda;
  const double* const* B; int64_t ldb;
  double* const* C; int64_t ldc;
  int batch;
};
hipError_t launch_zgemm(const ZUniformArgs& a, hipStream_t s);
// C_i <- beta C_i for complex C (beta == 0 writes exact zeros, C not read).
hipError_t launch_zscale(const double* beta, double* const* C, int64_t ldc, int m, int n,
                         int batch, hipStream_t s);

// Two-spin gates on batches of 2^S-amplitude states (in place).
hipError_t launch_gate2(int S, const int* sites, const double* const* U, double* const* psi,
                        int batch, int* info, hipStream_t s);

// Request loop: one generated factor (column-major n x n at `out`; factor j of
// `client`, values scaled by `scale`).
struct FillJob {   // 8-byte aligned, a multiple of 8 bytes: pointers may follow an array of them
  double* out;
  long long j;
  int n;
  int client;
  double scale;
};

// Generates the factors of njobs jobs (device array) in one launch; max_n is
// the largest n among them.
hipError_t launch_fill_factors(const FillJob* d_jobs, int njobs, int max_n,
                               unsigned long long seed, hipStream_t s);
// One factor, the same generator (host-side job).
hipError_t launch_fill_one(double* out, int n, int client, long long j, double scale,
                           unsigned long long seed, hipStream_t s);
// Annealing sweeps: factor t of a sweep for each job reads the client's
// product count at the start of the sweep from j0 (device) and uses
// j = j0[client] + t; k_advance adds `chain` to every j0 entry.
struct SweepJob {
  double* out;
  int n;
  int client;
  double scale;
};
hipError_t launch_fill_sweep(const SweepJob* d_jobs, int njobs, int max_n, const long long* d_j0,
                             int t, unsigned long long seed, hipStream_t s);
hipError_t launch_advance(long long* d_j0, int n, int chain, hipStream_t s);
// out <- identity (n x n, column-major, ld = n).
hipError_t launch_identity(double* out, int n, hipStream_t s);

}  // namespace bg
