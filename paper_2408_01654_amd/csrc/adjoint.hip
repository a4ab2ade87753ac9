// Adjoint of the unrolled Gauss-Newton iterations: gradients of a loss on
// the final poses and inverse depths with respect to the edge targets and
// confidence weights (the differentiable BA layer that supervises the
// predicted poses, Sec. 2; objective eq. 3).
//
// One iteration maps x_t = (poses, depths) to x_{t+1} = x_t (+) Delta with
// H~ Delta = -g, H~ = H + lam (Diag(H) + I), H = sum_e J_e^T W_e J_e and
// g = sum_e J_e^T W_e r_e over the free variables.  Walking the iterations
// backwards with the adjoint xbar of x_{t+1}:
//   1. retraction:  Deltabar = (dx_{t+1}/dDelta)^T xbar,  xbar_t = (dx_{t+1}/dx_t)^T xbar
//      (poses carry their adjoint in the stored (t, q) coordinates; the
//      differential of the retraction comes from dual-number evaluation);
//   2. solve:       u = H~^-1 Deltabar (Schur elimination with the stored
//      rows E_k / sqrt(C~_k), and a Cholesky solve of the reduced system),
//      so gbar = -u and H~bar = -u Delta^T;
//   3. damping:     Hbar = H~bar + lam Diag(H~bar);
//   4. per edge, on its 13 variables (xi_i, xi_j, d_k), per row c:
//        a_c = J_c u,  b_c = J_c Delta,
//        wbar_c   += -a_c b_c - lam sum_m J_cm^2 u_m Delta_m - r_c a_c,
//        taubar_c += w_c a_c            (r = pi - tau),
//        Jbar_c    = w_c (-(r_c + b_c) u - a_c Delta - 2 lam J_c o u o Delta),
//        rbar_c    = -w_c a_c;
//   5. xbar_t += d/dx [sum_c Jbar_c . J_c(x) + rbar_c r_c(x)] for the
//      coordinates (t_i, q_i, t_j, q_j, d_k), by walking the edge's evaluation
//      backwards (edge_pullback).
// Per-edge results are summed per pose and per patch in a fixed order.
#include <algorithm>

#include "dpvba.h"
#include "dual.h"
#include "edge.h"
#include "layout.h"
#include "tileargs.h"

namespace dpvba {

constexpr int kEdgeAdj = 15;  // (t_i, q_i) 7, (t_j, q_j) 7, d_k 1

// Rotation of a quaternion (x, y, z, w) with its unit quaternion u and the
// reciprocal norm n.
template <typename T>
__device__ __forceinline__ void unit_quat(const T* q, T u[4], T& n) {
  n = (T)1 / dsqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
  for (int m = 0; m < 4; ++m) u[m] = q[m] * n;
}

// Adjoint of quat_to_rot: B the adjoint of the rotation matrix, out [4] that
// of the stored quaternion (the component along it is projected out).
template <typename T>
__device__ __forceinline__ void rot_pullback(const T* q, const T B[9], T* out) {
  T u[4], n;
  unit_quat<T>(q, u, n);
  const T x = u[0], y = u[1], z = u[2], w = u[3];
  const T s01 = B[1] + B[3], s02 = B[2] + B[6], s12 = B[5] + B[7];
  const T d01 = B[3] - B[1], d02 = B[2] - B[6], d12 = B[7] - B[5];
  T g[4];
  g[0] = 2 * (y * s01 + z * s02 + w * d12) - 4 * x * (B[4] + B[8]);
  g[1] = 2 * (x * s01 + z * s12 + w * d02) - 4 * y * (B[0] + B[8]);
  g[2] = 2 * (x * s02 + y * s12 + w * d01) - 4 * z * (B[0] + B[4]);
  g[3] = 2 * (z * d01 + y * d02 + x * d12);
  const T dot = x * g[0] + y * g[1] + z * g[2] + w * g[3];
  for (int m = 0; m < 4; ++m) out[m] = n * (g[m] - u[m] * dot);
}

// Gradient of sum_c Jb_c . J_c + rb_c r_c with respect to the stored (t, q)
// of both poses and the depth, xb [15]: the steps of the edge's evaluation
// (edge_eval, the source pose's Jacobian, relative_pose, quat_to_rot) in
// reverse.  Ri, Rj, Rt: the rotations and the relative pose; o: the edge's
// terms.  (J is the 2 x 13 (J_i | J_j | J_d).)
template <typename T>
__device__ __forceinline__ void edge_pullback(const T* pi, const T* pj, const T Ri[9], const T Rj[9], const T Rt[12],
                                              const EdgeTerms<T>& o, T d, T xh0, T xh1, T fx, T fy, const T rb[2],
                                              const T Jb[2][13], T* xb) {
  const T *R = Rt, *t = Rt + 9;
  T Rb[9], tb[3], G[2][6];
  for (int m = 0; m < 9; ++m) Rb[m] = (T)0;
  for (int m = 0; m < 3; ++m) tb[m] = (T)0;
  for (int c = 0; c < 2; ++c) {  // J_i = -(R^T a ; R^T (b - t x a)) of J_j = (a ; b)
    const T* a = o.Jj[c];
    const T b[3] = {a[3] - (t[1] * a[2] - t[2] * a[1]), a[4] - (t[2] * a[0] - t[0] * a[2]),
                    a[5] - (t[0] * a[1] - t[1] * a[0])};
    const T* g = Jb[c];  // o1 = -g[0..2], o2 = -g[3..5]
    T bb[3];
    for (int r = 0; r < 3; ++r) bb[r] = -(R[3 * r] * g[3] + R[3 * r + 1] * g[4] + R[3 * r + 2] * g[5]);
    for (int r = 0; r < 3; ++r)
      for (int k = 0; k < 3; ++k) Rb[3 * r + k] -= a[r] * g[k] + b[r] * g[3 + k];
    // -bb . (t x a): to t -(a x bb), to a -(bb x t)
    tb[0] -= a[1] * bb[2] - a[2] * bb[1];
    tb[1] -= a[2] * bb[0] - a[0] * bb[2];
    tb[2] -= a[0] * bb[1] - a[1] * bb[0];
    for (int r = 0; r < 3; ++r) {
      const T ra = -(R[3 * r] * g[0] + R[3 * r + 1] * g[1] + R[3 * r + 2] * g[2]);
      const T bt = bb[(r + 1) % 3] * t[(r + 2) % 3] - bb[(r + 2) % 3] * t[(r + 1) % 3];
      G[c][r] = g[6 + r] + ra - bt;
      G[c][3 + r] = g[9 + r] + bb[r];
    }
  }
  const T q0 = R[0] * xh0 + R[1] * xh1 + R[2] + t[0] * d;
  const T q1 = R[3] * xh0 + R[4] * xh1 + R[5] + t[1] * d;
  const T q2 = R[6] * xh0 + R[7] * xh1 + R[8] + t[2] * d;
  const T iz = (T)1 / q2;
  const T ax0 = fx * iz, ax2 = -fx * q0 * iz * iz, by1 = fy * iz, by2 = -fy * q1 * iz * iz;
  const T gd0 = Jb[0][12], gd1 = Jb[1][12];
  const T ax0b = -d * G[0][0] - q2 * G[0][4] + q1 * G[0][5] + t[0] * gd0;
  const T ax2b = -d * G[0][2] - q1 * G[0][3] + q0 * G[0][4] + t[2] * gd0;
  const T by1b = -d * G[1][1] + q2 * G[1][3] - q0 * G[1][5] + t[1] * gd1;
  const T by2b = -d * G[1][2] - q1 * G[1][3] + q0 * G[1][4] + t[2] * gd1;
  T db = -ax0 * G[0][0] - ax2 * G[0][2] - by1 * G[1][1] - by2 * G[1][2];
  tb[0] += ax0 * gd0;
  tb[1] += by1 * gd1;
  tb[2] += ax2 * gd0 + by2 * gd1;
  T qb[3] = {ax2 * G[0][4] + by2 * G[1][4] - by1 * G[1][5], ax0 * G[0][5] - ax2 * G[0][3] - by2 * G[1][3],
             by1 * G[1][3] - ax0 * G[0][4]};
  const T iz2 = iz * iz;
  const T izb = fx * (q0 * rb[0] + ax0b - 2 * q0 * iz * ax2b) + fy * (q1 * rb[1] + by1b - 2 * q1 * iz * by2b);
  qb[0] += fx * (iz * rb[0] - iz2 * ax2b);
  qb[1] += fy * (iz * rb[1] - iz2 * by2b);
  qb[2] -= iz2 * izb;
  const T xh[3] = {xh0, xh1, (T)1};
  for (int r = 0; r < 3; ++r) {
    for (int k = 0; k < 3; ++k) Rb[3 * r + k] += qb[r] * xh[k];
    tb[r] += d * qb[r];
    db += t[r] * qb[r];
  }
  // R = R_j^T R_i, t = R_j^T (t_i - t_j)
  T Rib[9], Rjb[9];
  for (int k = 0; k < 3; ++k) {
    const T dk = pi[k] - pj[k];
    T s = (T)0;
    for (int r = 0; r < 3; ++r) {
      Rib[3 * k + r] = Rj[3 * k] * Rb[r] + Rj[3 * k + 1] * Rb[3 + r] + Rj[3 * k + 2] * Rb[6 + r];
      Rjb[3 * k + r] = Rb[3 * r] * Ri[3 * k] + Rb[3 * r + 1] * Ri[3 * k + 1] + Rb[3 * r + 2] * Ri[3 * k + 2] + tb[r] * dk;
      s += Rj[3 * k + r] * tb[r];
    }
    xb[k] = s;
    xb[7 + k] = -s;
  }
  rot_pullback<T>(pi + 3, Rib, xb + 3);
  rot_pullback<T>(pj + 3, Rjb, xb + 10);
  xb[14] = db;
}

// Start of the walk: cleared status words, x_0, and the adjoint of x_T in
// tile order (zero without one).
template <typename T>
__global__ void __launch_bounds__(256) adj_begin_kernel(AdjGroup<T> G) {
  const AdjArgs<T>& a = G.p[blockIdx.y];
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < 2 * DPVBA_MAX_ITERS) {
    a.status[q] = 0;
    a.mb[q] = 0x7f7fffffu;  // bits of FLT_MAX
  }
  if (q == 0) *a.it.dev_err = 0;
  if (q < 7 * a.it.n_frames) {
    a.Xp[q] = a.poses0[q];
    a.pbar[q] = a.grad_poses ? a.grad_poses[q] : (T)0;
  }
  if (q < a.n_tp) a.dbar[q] = a.grad_depth ? a.grad_depth[a.it.tile_patch[q]] : (T)0;
}

// Steps 4 and 5 for every edge.  u and Delta of the poses are indexed by free
// pose, of the depths by tile-order position.  Adds taubar and wbar to the
// caller's gradients (the walk's first iteration, the last one, stores them)
// and writes the edge's xbar contributions.  Bound by an edge's dependent
// arithmetic and its 120 scattered bytes; the reverse walk is about three
// evaluations of the edge, where a dual evaluation for each of the 15
// coordinates took 29.4 us for a float64 window of 22 frames, this 11.4 us.
template <typename T>
__global__ void __launch_bounds__(128) edge_adjoint_kernel(AdjGroup<T> G, int it) {
  const AdjArgs<T>& a = G.p[blockIdx.y];
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n_edges) return;
  const bool first = it == a.nit - 1;
  const int n_fixed = a.it.n_fixed, p = a.it.p;
  const T *poses = a.Xp + (size_t)it * 7 * a.it.n_frames, *dxi = a.DX + (size_t)it * 6 * a.it.n_free;
  const T fx = a.it.fx, fy = a.it.fy, cx = a.it.cx, cy = a.it.cy, lam_diag = a.it.lam_diag;
  T* xb = a.exb + (size_t)kEdgeAdj * e;
  const bool skip = a.status[it] != 0;
  const int i = a.ii[e], j = a.jj[e], k = a.kk[e];
  const int pos = a.patch_pos[k];
  const int c0 = (p - 1) / 2;
  const float* cen = a.it.patches + ((size_t)k * p * p + (size_t)c0 * p + c0) * 2;
  const T xh0 = ((T)cen[0] - cx) / fx, xh1 = ((T)cen[1] - cy) / fy;
  T pi[7], pj[7];
  for (int m = 0; m < 7; ++m) {
    pi[m] = poses[7 * (size_t)i + m];
    pj[m] = poses[7 * (size_t)j + m];
  }
  const T d = a.Xd[(size_t)it * a.n_tp + pos];
  const float w0 = a.it.weight[2 * e], w1 = a.it.weight[2 * e + 1];
  T Ri[9], Rj[9], Rt[12];
  quat_to_rot<T, T>(pi + 3, Ri);
  quat_to_rot<T, T>(pj + 3, Rj);
  relative_pose<T>(Ri, pi, Rj, pj, Rt, Rt + 9);
  EdgeTerms<T> o;
  const bool ok = !skip && edge_eval<T>(Rt, xh0, xh1, d, fx, fy, cx, cy, a.it.z_min, a.it.target[2 * e],
                                        a.it.target[2 * e + 1], w0, w1, o);
  if (!ok) {
    for (int m = 0; m < kEdgeAdj; ++m) xb[m] = (T)0;
    if (first)
      for (int c = 0; c < 2; ++c) {
        a.grad_weight[2 * e + c] = (T)0;
        a.grad_target[2 * e + c] = (T)0;
      }
    return;
  }
  const bool fi = i >= n_fixed, fj = j >= n_fixed;
  T u[13], D[13];
  for (int m = 0; m < 6; ++m) {
    u[m] = fi ? a.up[6 * (i - n_fixed) + m] : (T)0;
    D[m] = fi ? dxi[6 * (i - n_fixed) + m] : (T)0;
    u[6 + m] = fj ? a.up[6 * (j - n_fixed) + m] : (T)0;
    D[6 + m] = fj ? dxi[6 * (j - n_fixed) + m] : (T)0;
  }
  u[12] = a.ud[pos];
  D[12] = a.dd[pos];
  T Jb[2][13], rb[2];
  for (int c = 0; c < 2; ++c) {
    T J[13], ji[6];
    adjoint_transpose_apply<T>(Rt, Rt + 9, o.Jj[c], ji);
    for (int m = 0; m < 6; ++m) {
      J[m] = -ji[m];
      J[6 + m] = o.Jj[c][m];
    }
    J[12] = o.Jd[c];
    const T w = o.w[c];
    T av = (T)0, b = (T)0, sd = (T)0;
    for (int m = 0; m < 13; ++m) {
      av += J[m] * u[m];
      b += J[m] * D[m];
      sd += J[m] * J[m] * u[m] * D[m];
    }
    const T gw = -av * b - lam_diag * sd - o.r[c] * av, gt = w * av;
    a.grad_weight[2 * e + c] = first ? gw : a.grad_weight[2 * e + c] + gw;
    a.grad_target[2 * e + c] = first ? gt : a.grad_target[2 * e + c] + gt;
    rb[c] = -w * av;
    for (int m = 0; m < 13; ++m)
      Jb[c][m] = w * (-(o.r[c] + b) * u[m] - av * D[m] - (T)2 * lam_diag * J[m] * u[m] * D[m]);
  }
  T x[kEdgeAdj];
  edge_pullback<T>(pi, pj, Ri, Rj, Rt, o, d, xh0, xh1, fx, fy, rb, Jb, x);
  for (int m = 0; m < kEdgeAdj; ++m) xb[m] = (m < 7 && !fi) || (m >= 7 && m < 14 && !fj) ? (T)0 : x[m];
}

// Step 2, first half: per tile and block column x, the tile's share of
// -E C~^-1 Deltabar_d = -sum_k U_kx (1 / sqrt(C~_k)) Deltabar_d,k, written to
// the right-hand-side part of the tile's partial vector.  The rows go to as
// many groups of threads as fit beside the columns.
template <typename T>
__global__ void __launch_bounds__(256) tile_adjoint_rhs_kernel(AdjGroup<T> G) {
  __shared__ T sc[256], red[256];
  const AdjArgs<T>& a = G.p[blockIdx.y];
  if ((int)blockIdx.x >= a.it.n_tiles) return;
  const TileInfo ti = a.it.tiles[blockIdx.x];
  const int W6 = 6 * ti.n_blk, Ws = tile_u_stride(ti.n_blk), tid = threadIdx.x;
  const T* U = a.it.U_s + ti.u_begin;
  const int ng = W6 > 0 && W6 <= 128 ? 256 / W6 : 1, grp = ng > 1 ? tid / W6 : 0;
  for (int x = ng > 1 ? tid - grp * W6 : tid;; x += 256) {  // one pass when W6 <= 256
    const bool on = grp < ng && x < W6;
    T v = (T)0;
    for (int k0 = 0; k0 < ti.n_patch; k0 += 256) {
      __syncthreads();
      if (k0 + tid < ti.n_patch) {
        const int q = ti.patch_begin + k0 + tid;
        sc[tid] = a.it.pscale_s[2 * q] * a.dbar[q];
      }
      __syncthreads();
      const int kn = min(256, ti.n_patch - k0);
      if (on) {
#pragma unroll 8
        for (int k = grp; k < kn; k += ng) v += U[(size_t)(k0 + k) * Ws + x] * sc[k];
      }
    }
    if (ng > 1) {
      red[tid] = v;
      __syncthreads();
      if (tid < W6) {
        v = (T)0;
        for (int h = 0; h < ng; ++h) v += red[h * W6 + tid];
        a.it.part_vec[ti.vec_begin + tid] = -v;
      }
    } else if (on) {
      a.it.part_vec[ti.vec_begin + x] = -v;
    }
    if (ng > 1 || x - tid + 256 >= W6) break;  // uniform
  }
}

// rhs = Deltabar_xi + the tiles' shares, summed per free pose in tile order.
template <typename T>
__global__ void vec_gather_add_kernel(const T* part_vec, const int* off, const int2* src, int n, const T* add,
                                      const int* status, T* out) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const int P_ = x / 6, m = x % 6;
  T v = add[x];
  for (int q = off[P_]; q < off[P_ + 1]; ++q) v += part_vec[src[q].x + m];
  out[x] = (status && *status) ? (T)0 : v;
}

// Step 2, second half, per patch of a tile: the depth part of u,
// u_d = C~^-1 (Deltabar_d - E^T u_p), and the forward depth step
// Delta_d = C~^-1 (-w - E^T Delta_xi), both from the stored rows.
template <typename T>
__global__ void __launch_bounds__(256) tile_adjoint_backsub_kernel(AdjGroup<T> G, int it) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T* sU = reinterpret_cast<T*>(lds_raw);
  const AdjArgs<T>& a = G.p[blockIdx.y];
  if ((int)blockIdx.x >= a.it.n_tiles) return;
  const TileInfo ti = a.it.tiles[blockIdx.x];
  const int W6 = 6 * ti.n_blk, Ws = tile_u_stride(ti.n_blk);
  const T* dxi = a.DX + (size_t)it * 6 * a.it.n_free;
  T* sX = sU + W6;
  for (int x = threadIdx.x; x < W6; x += blockDim.x) {
    const int f = a.it.blk_pose[ti.blk_begin + x / 6];
    sU[x] = a.up[6 * f + x % 6];
    sX[x] = dxi[6 * f + x % 6];
  }
  __syncthreads();
  const bool skip = a.status[it] != 0;
  const T* U = a.it.U_s + ti.u_begin;
  for (int k = threadIdx.x; k < ti.n_patch; k += blockDim.x) {
    const int q = ti.patch_begin + k;
    const T is = a.it.pscale_s[2 * q], rs = a.it.pscale_s[2 * q + 1];
    T du = (T)0, dx = (T)0;
    for (int x = 0; x < W6; ++x) {
      const T uk = U[(size_t)k * Ws + x];
      du += uk * sU[x];
      dx += uk * sX[x];
    }
    a.ud[q] = skip ? (T)0 : is * (a.dbar[q] * is - du);
    a.dd[q] = skip ? (T)0 : -(rs + dx) * is;
  }
}

// Step 5 sums of iteration it + 1, then step 1 of iteration `it` (either left
// out at the ends of the walk: it = nit - 1, it = -1).  Workgroups below the
// number of free poses take one pose each: xbar gets its edges' shares (pose_src
// holds 2 e + side, side 0 = source, 1 = target), thread t the list entries
// t, t + 256, ..., and the partial sums are combined by a fixed tree, so the
// result does not depend on timing; then the adjoint before the retraction
// and that of its step, one coordinate a thread (one thread a pose took 28 us
// for the 13 dual evaluations).  The other workgroups sum the depths, per
// tile-order patch position its edges in edge order.
template <typename T>
__global__ void __launch_bounds__(256) adj_reduce_kernel(AdjGroup<T> G, int it) {
  __shared__ T red[7][256];
  const AdjArgs<T>& a = G.p[blockIdx.y];
  const int n_free = a.it.n_free, tid = threadIdx.x;
  const bool sum = it + 1 < a.nit;
  if ((int)blockIdx.x >= n_free) {
    const int q = ((int)blockIdx.x - n_free) * 256 + tid;
    if (!sum || q >= a.n_tp) return;
    const int k = a.it.tile_patch[q], hi = a.pcount[k + 1];
    T v = (T)0;
    for (int lo = a.pcount[k]; lo < hi; lo += 8) {
      T x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        x[u] = a.exb[(size_t)kEdgeAdj * a.pedges[min(lo + u, hi - 1)] + 14];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += lo + u < hi ? x[u] : (T)0;
    }
    a.dbar[q] += v;
    return;
  }
  const int f = a.it.n_fixed + blockIdx.x, fr = blockIdx.x;
  T* pb = a.pbar + 7 * (size_t)f;
  T* out_bar = red[0];
  if (sum) {
    T v[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int q = a.pose_off[f] + tid; q < a.pose_off[f + 1]; q += 256) {
      const int s = a.pose_src[q];
      const T* x = a.exb + (size_t)kEdgeAdj * (s >> 1) + 7 * (s & 1);
#pragma unroll
      for (int m = 0; m < 7; ++m) v[m] += x[m];
    }
#pragma unroll
    for (int m = 0; m < 7; ++m) red[m][tid] = v[m];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if (tid < w)
#pragma unroll
        for (int m = 0; m < 7; ++m) red[m][tid] += red[m][tid + w];
      __syncthreads();
    }
  }
  T pv = (T)0;
  if (tid < 7) pv = sum ? pb[tid] + red[tid][0] : pb[tid];
  __syncthreads();
  if (tid < 7) out_bar[tid] = pv;
  __syncthreads();
  const bool skip = it < 0 || a.status[it] != 0;  // a skipped iteration is the identity map
  if (skip) {
    if (tid < 7) pb[tid] = pv;
    if (it >= 0 && tid < 6) a.dxbar[6 * fr + tid] = (T)0;
    return;
  }
  if (tid >= 13) return;
  const T* x = a.Xp + ((size_t)it * a.it.n_frames + f) * 7;
  const T* s = a.DX + ((size_t)it * n_free + fr) * 6;
  using D1 = Dual<T>;
  D1 pose[7], xi[6];
  for (int m = 0; m < 7; ++m) pose[m] = D1(x[m], tid == m ? (T)1 : (T)0);
  for (int m = 0; m < 6; ++m) xi[m] = D1(s[m], tid == 7 + m ? (T)1 : (T)0);
  retract_pose<D1, D1>(pose, xi);
  T acc = (T)0;
  for (int m = 0; m < 7; ++m) acc += out_bar[m] * pose[m].d;
  if (tid < 7) pb[tid] = acc;
  else a.dxbar[6 * fr + tid - 7] = acc;
}

template <typename T>
__global__ void fill_kernel(T* x, long long n, T v) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n) x[q] = v;
}

// ---------------------------------------------------------------- launchers

static inline unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// G holds n problems; the sizes are their largest.
template <typename T>
hipError_t launch_adj_begin(const AdjGroup<T>& G, int n, int n_frames, int n_tp, hipStream_t st) {
  const int m = std::max(std::max(7 * n_frames, n_tp), 2 * DPVBA_MAX_ITERS);
  hipLaunchKernelGGL((adj_begin_kernel<T>), dim3(blocks_for(m, 256), n), dim3(256), 0, st, G);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_edge_adjoint(const AdjGroup<T>& G, int n, int n_edges, int it, hipStream_t st) {
  if (n_edges == 0) return hipSuccess;
  hipLaunchKernelGGL((edge_adjoint_kernel<T>), dim3(blocks_for(n_edges, 128), n), dim3(128), 0, st, G, it);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adjoint_rhs(const AdjGroup<T>& G, int n, int n_tiles, hipStream_t st) {
  if (n_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL((tile_adjoint_rhs_kernel<T>), dim3(n_tiles, n), dim3(256), 0, st, G);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_vec_gather_add(const T* part_vec, const int* v_off, const int2* v_src, int n_free, const T* add,
                                 const int* status, T* out, hipStream_t st) {
  const int n = 6 * n_free;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL((vec_gather_add_kernel<T>), dim3(blocks_for(n, 256)), dim3(256), 0, st, part_vec, v_off, v_src, n,
                     add, status, out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adjoint_backsub(const AdjGroup<T>& G, int n, int n_tiles, int max_w6, int it, hipStream_t st) {
  if (n_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL((tile_adjoint_backsub_kernel<T>), dim3(n_tiles, n), dim3(256), 2 * max_w6 * (int)sizeof(T), st, G,
                     it);
  return hipGetLastError();
}

// Sums of iteration it + 1 (blocks of the largest problem: n_free poses and
// n_tp depths; a smaller problem's depths start after its own poses) and the
// retraction's adjoint of iteration `it`.
template <typename T>
hipError_t launch_adj_reduce(const AdjGroup<T>& G, int n, int n_free, int n_tp, int it, hipStream_t st) {
  const unsigned blocks = (unsigned)n_free + blocks_for(n_tp, 256);
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((adj_reduce_kernel<T>), dim3(blocks, n), dim3(256), 0, st, G, it);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_fill(T* x, long long n, T v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL((fill_kernel<T>), dim3(blocks_for(n, 256)), dim3(256), 0, st, x, n, v);
  return hipGetLastError();
}

#define DPVBA_ADJ_INST(T)                                                                                        \
  template hipError_t launch_adj_begin<T>(const AdjGroup<T>&, int, int, int, hipStream_t);                       \
  template hipError_t launch_edge_adjoint<T>(const AdjGroup<T>&, int, int, int, hipStream_t);                    \
  template hipError_t launch_adjoint_rhs<T>(const AdjGroup<T>&, int, int, hipStream_t);                          \
  template hipError_t launch_vec_gather_add<T>(const T*, const int*, const int2*, int, const T*, const int*, T*, \
                                               hipStream_t);                                                     \
  template hipError_t launch_adjoint_backsub<T>(const AdjGroup<T>&, int, int, int, int, hipStream_t);            \
  template hipError_t launch_adj_reduce<T>(const AdjGroup<T>&, int, int, int, int, hipStream_t);                 \
  template hipError_t launch_fill<T>(T*, long long, T, hipStream_t);
DPVBA_ADJ_INST(float)
DPVBA_ADJ_INST(double)
template hipError_t launch_fill<int>(int*, long long, int, hipStream_t);
#undef DPVBA_ADJ_INST

}  // namespace dpvba
