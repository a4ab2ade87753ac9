// Device view of a block elimination plan (blockplan.h) and the launchers of
// the kernels that follow it (sparse.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "blockplan.h"

namespace dpvba {

// Lists of a plan on the device (host arrays where said), by value into the
// launchers.
struct SparsePlan {
  int bw, n_pose, nb, n_level, n_blocks;
  const int* row0;      // per pose: first row in the padded vectors (64 nb rows)
  const int* size;      // rows used of each block
  const int* colptr;    // block ids of each block column, diagonal first
  const int* rowidx;    // block row of each id
  const int* level;     // per block column
  const LevelTask* tasks;
  const LevelChild* children;
  const UpdateTask* updates;
  const UpdateSrc* srcs;
  const int* by_level;  // block columns by level
  const int* rptr;      // each block row's columns: rlist[rptr[I] .. rptr[I + 1])
  const int2* rlist;    // (J, id) by level
  // original (unfilled) blocks of the symmetric matrix by block row: (other
  // block, 2 id + 1 if it is used transposed)
  const int* nptr;
  const int2* nlist;
  // gather of the tiles' shares: each block's pose pairs, x = share list,
  // y = first row | first column << 8 | transposed << 16 | diagonal pair << 17
  const int* pair_off;
  const int2* pairs;
  // host
  const int* task_off;
  const int* upd_off;
  const int* implicit_col;
  const int* colptr_h;
};

// A <- the damped reduced system in block storage from the tiles' shares
// (part_S, share lists off / src), identity on unused rows; d0 [64 nb] its
// diagonal; dB [64 nb] Diag(B) (gathered before); rhs [64 nb]: its unused rows
// are zeroed.  A32: optional float32 copy of A (and d032 of d0).
template <typename TP, typename T>
hipError_t launch_sparse_gather(const SparsePlan& p, const TP* part_S, const int* off, const int* src, T* A,
                                const T* dB, T lambda, T lam_diag, T* d0, T* rhs, float* A32, float* d032,
                                hipStream_t st);
// A <- zero blocks with identity on unused rows; v [64 nb] <- zero; *cost (if
// given) <- the sum of the squares of r [nr].
template <typename T>
hipError_t launch_sparse_clear(const SparsePlan& p, T* A, T* v, const double* r, int nr, double* cost,
                               hipStream_t st);
// A <- its Cholesky factor (off-diagonal blocks; the diagonal blocks keep
// their input), Linv [nb][64][64] the inverses of the factor's diagonal
// blocks, v <- L^-1 v.  *status is set by a pivot that is not positive,
// *min_bits receives the smallest L_ii^2 / S_ii.
template <typename T>
hipError_t launch_sparse_factor(const SparsePlan& p, T* A, T* Linv, T* v, const T* d0, int* status,
                                unsigned int* min_bits, hipStream_t st);
// x = L^-T y (backward_only) or x = (L L^T)^-1 b with y as work space.
template <typename T>
hipError_t launch_sparse_solve(const SparsePlan& p, const T* A, const T* Linv, const T* b, T* y, T* x,
                               unsigned long long* words, int epoch, int* err, int* host_err, hipStream_t st,
                               bool backward_only, bool cooperative, const unsigned long long* stop = nullptr,
                               double tol = 0.0);
// Refined solve of the unfactored system: y = fl32(s) and n_res pairs of maxima
// cleared; then x_out = x_in + c (x_in null: c alone; without c when the
// residual before, stop, is at or below tol), rhs = fl32(s - A x_out), maxes
// [0], [1]: largest |r|, |s|.
hipError_t launch_sparse_refine_begin(const SparsePlan& p, const double* s, float* y, unsigned long long* maxes,
                                      int n_res, hipStream_t st);
hipError_t launch_sparse_residual(const SparsePlan& p, const double* A, const double* s, const double* x_in,
                                  const float* c, const unsigned long long* stop, double tol, double* x_out, float* rhs,
                                  unsigned long long* maxes, hipStream_t st);
// Rows of the poses (bw each) into the padded order (zero elsewhere) and out
// of it; out of it with *status set: zero.
template <typename T>
hipError_t launch_sparse_rows_in(const SparsePlan& p, const T* src, T* dst, hipStream_t st);
template <typename T>
hipError_t launch_sparse_rows_out(const SparsePlan& p, const T* src, T* dst, const int* status, hipStream_t st);

// 64-bit words of the solve's published values: two passes, two words a row.
inline size_t sparse_words_bytes(size_t nb) { return 2 * nb * kBlk * 2 * 8; }

}  // namespace dpvba
