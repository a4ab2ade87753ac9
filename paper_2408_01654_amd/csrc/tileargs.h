// Arguments of the tile kernels and of the single-launch small-problem solver.
#pragma once

#include <hip/hip_runtime.h>

#include "layout.h"

namespace dpvba {

template <typename T>
struct IterArgs {
  const float* patches;
  int p;
  const float* target;
  const float* weight;
  T fx, fy, cx, cy, z_min;
  T lambda;                // additive damping: H~ = H + lam_diag Diag(H) + lambda I
  T lam_diag;              // lambda (Levenberg-Marquardt) or 0 (Levenberg)
  int n_frames, n_fixed, n_free, n_tiles;
  const T* poses_cur;      // [N,7] x_t
  T* poses_next;           // [N,7] x_{t+1} (written by the last workgroup)
  const T* depth_in;       // caller's inverse depths (read when first)
  T* depth_s;              // tile-ordered inverse depths (written)
  const T* depth_prev;     // those of the step before (depth_s, or an array of its own)
  T* xh_s;                 // tile-ordered patch rays [.,2]
  T* U_s;                  // stored Schur rows
  T* pscale_s;             // per patch: 1/sqrt(C~), w/sqrt(C~)
  const T* dx_prev;        // previous pose step (applied unless first)
  const int* status_prev;  // nonzero: previous step discarded (entry inst * status_stride)
  int status_stride;       // distance between the problems' status words (0: one problem)
  int first;
  const TileInfo* tiles;
  const int* tile_patch;
  const int* slot_frame;
  const int* slot_blk;
  const int* edge_grid;
  const int* blk_pose;
  T* part_S;
  T* part_vec;
  double* part_cost;
  int* part_invalid;
  // gather lists and per-iteration outputs of the small-problem solver
  const int* s_off;
  const int* s_src;
  const int* v_off;
  const int2* v_src;
  T* dx;
  int* status;
  unsigned int* min_bits;
  double* cost_out;
  int* invalid_out;
  int* dev_err;            // device failure word of the call (bit 4: invalid target / weight)
  int* host_err;           // host-visible sticky copy of the failure bits
  const int* order;        // one launch per pass: workgroup g runs tile order[g] (heaviest first), or g if null
};

// Arguments of the single-launch solver of small problems.
template <typename T>
struct SmallArgs {
  IterArgs<T> it;       // shared fields; per-iteration fields set in the kernel
  T* poses_io;          // caller's poses (read at t = 0, written at the end)
  T* depth_io;          // caller's inverse depths
  T* pbuf0;
  T* pbuf1;
  T* Sp;                // packed reduced system
  T* rhs;
  T* d0;
  int* status;          // per iteration
  unsigned int* min_bits;
  double* cost;         // per iteration, or null
  int* invalid;
  int n_iters;
  unsigned int* bar;       // this launch's grid-barrier slot (arrivals, generation)
  unsigned int* bar_next;  // the next launch's slot, cleared by this one
  int* err;                // this launch's failure word
  int* err_next;           // the next launch's failure word, cleared by this one
};

// Several small problems side by side: every launch takes up to kSmallGroup,
// blockIdx.y.  Passed by value, so it has to fit the 4 KB of a kernel's
// arguments.
constexpr int kSmallGroup = 8;
template <typename T>
struct SmallGroup {
  SmallArgs<T> p[kSmallGroup];
};
static_assert(sizeof(SmallGroup<double>) + 64 <= 4096, "kernel arguments");

// One problem of an adjoint launch: every launch of the adjoint takes up to
// kAdjGroup problems, blockIdx.y (by value, within the 4 KB of a kernel's
// arguments).  X and D hold the replayed iterates and steps, one after another.
template <typename T>
struct AdjArgs {
  IterArgs<T> it;      // tile arguments; per-iteration fields set in the kernels (adj_iter)
  int nit, n_edges, n_tp;
  T* Xp;               // [nit + 1][N, 7] poses
  T* Xd;               // [nit][n_tp] inverse depths, tile order
  T* DX;               // [nit][6 n_free] steps
  T *pbar, *dbar;      // adjoint of the poses [N, 7] and of the depths (tile order)
  T *dxbar, *urhs;     // adjoint of the step, right-hand side of the solve
  T *up, *ud, *dd;     // u = H~^-1 Deltabar (poses, depths), depth steps
  T* exb;              // per edge: its 15 shares of the adjoint
  int* status;         // [2 DPVBA_MAX_ITERS]: replayed steps, adjoint solves
  unsigned int* mb;
  T *Sp, *rhs, *d0;    // damped reduced system (packed for the small solver)
  const T *poses0, *grad_poses, *grad_depth;
  T *grad_target, *grad_weight;
  const int *ii, *jj, *kk, *patch_pos, *pose_off, *pose_src, *pcount, *pedges;
};
constexpr int kAdjGroup = 6;
template <typename T>
struct AdjGroup {
  AdjArgs<T> p[kAdjGroup];
};
static_assert(sizeof(AdjGroup<double>) + 64 <= 4096, "kernel arguments");

}  // namespace dpvba
