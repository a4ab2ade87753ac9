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
//   5. xbar_t += d/dx [sum_c Jbar_c . J_c(x) + rbar_c r_c(x)], one dual
//      evaluation of the edge per coordinate of (t_i, q_i, t_j, q_j, d_k).
// Per-edge results are summed per pose and per patch in a fixed order.
#include <algorithm>

#include "dpvba.h"
#include "dual.h"
#include "edge.h"
#include "layout.h"
#include "tileargs.h"

namespace dpvba {

constexpr int kEdgeAdj = 15;  // (t_i, q_i) 7, (t_j, q_j) 7, d_k 1

// Residual and the 2 x 13 Jacobian (J_i | J_j | J_d) of one edge at poses
// (t, q) of frames i and j and inverse depth d; false if the edge is invalid.
template <typename T>
__device__ __forceinline__ bool edge_full(const T* pi, const T* pj, T d, T xh0, T xh1, T fx, T fy, T cx, T cy,
                                          T z_min, float tx, float ty, T r[2], T J[2][13]) {
  T Ri[9], Rj[9], ti[3], tj[3], Rt[12];
  quat_to_rot<T, T>(pi + 3, Ri);
  quat_to_rot<T, T>(pj + 3, Rj);
  for (int m = 0; m < 3; ++m) { ti[m] = pi[m]; tj[m] = pj[m]; }
  relative_pose<T>(Ri, ti, Rj, tj, Rt, Rt + 9);
  EdgeTerms<T> o;
  if (!edge_eval<T>(Rt, xh0, xh1, d, fx, fy, cx, cy, z_min, tx, ty, 1.f, 1.f, o)) return false;
  for (int c = 0; c < 2; ++c) {
    T ji[6];
    adjoint_transpose_apply<T>(Rt, Rt + 9, o.Jj[c], ji);
    for (int m = 0; m < 6; ++m) {
      J[c][m] = -ji[m];
      J[c][6 + m] = o.Jj[c][m];
    }
    J[c][12] = o.Jd[c];
    r[c] = o.r[c];
  }
  return true;
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
// and writes the edge's xbar contributions.  Bound by the dependent
// arithmetic of the 15 dual evaluations: four lanes share an edge, so a
// window's 20 thousand edges fill the SIMDs (@E@).
template <typename T>
__global__ void __launch_bounds__(256) edge_adjoint_kernel(AdjGroup<T> G, int it) {
  const AdjArgs<T>& a = G.p[blockIdx.y];
  const int e = (blockIdx.x * blockDim.x + threadIdx.x) >> 2, part = threadIdx.x & 3;
  if (e >= a.n_edges) return;
  const bool first = it == a.nit - 1;
  const int n_fixed = a.it.n_fixed, p = a.it.p;
  const T *poses = a.Xp + (size_t)it * 7 * a.it.n_frames, *dxi = a.DX + (size_t)it * 6 * a.it.n_free;
  const T fx = a.it.fx, fy = a.it.fy, cx = a.it.cx, cy = a.it.cy, z_min = a.it.z_min, lam_diag = a.it.lam_diag;
  T* xb = a.exb + (size_t)kEdgeAdj * e;
  const bool skip = a.status[it] != 0;
  const int i = a.ii[e], j = a.jj[e], k = a.kk[e];
  const int pos = a.patch_pos[k];
  const int c0 = (p - 1) / 2;
  const float* cen = a.it.patches + ((size_t)k * p * p + (size_t)c0 * p + c0) * 2;
  const T xh0 = ((T)cen[0] - cx) / fx, xh1 = ((T)cen[1] - cy) / fy;
  const T* pi = poses + 7 * (size_t)i;
  const T* pj = poses + 7 * (size_t)j;
  const T d = a.Xd[(size_t)it * a.n_tp + pos];
  const float tx = a.it.target[2 * e], ty = a.it.target[2 * e + 1];
  T r[2], J[2][13];
  const bool ok = !skip && edge_full<T>(pi, pj, d, xh0, xh1, fx, fy, cx, cy, z_min, tx, ty, r, J);
  if (!ok) {
    for (int m = part; m < kEdgeAdj; m += 4) xb[m] = (T)0;
    if (first && part < 2) {
      a.grad_weight[2 * e + part] = (T)0;
      a.grad_target[2 * e + part] = (T)0;
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
    const T w = (T)a.it.weight[2 * e + c];
    T av = (T)0, b = (T)0, sd = (T)0;
    for (int m = 0; m < 13; ++m) {
      av += J[c][m] * u[m];
      b += J[c][m] * D[m];
      sd += J[c][m] * J[c][m] * u[m] * D[m];
    }
    if (part == 0) {
      const T gw = -av * b - lam_diag * sd - r[c] * av, gt = w * av;
      a.grad_weight[2 * e + c] = first ? gw : a.grad_weight[2 * e + c] + gw;
      a.grad_target[2 * e + c] = first ? gt : a.grad_target[2 * e + c] + gt;
    }
    rb[c] = -w * av;
    for (int m = 0; m < 13; ++m)
      Jb[c][m] = w * (-(r[c] + b) * u[m] - av * D[m] - (T)2 * lam_diag * J[c][m] * u[m] * D[m]);
  }
  // directional derivatives of (r, J) along each stored coordinate
  using D1 = Dual<T>;
  for (int dir = part; dir < kEdgeAdj; dir += 4) {
    if ((dir < 7 && !fi) || (dir >= 7 && dir < 14 && !fj)) {
      xb[dir] = (T)0;
      continue;
    }
    D1 Pi[7], Pj[7];
    for (int m = 0; m < 7; ++m) {
      Pi[m] = D1(pi[m], dir == m ? (T)1 : (T)0);
      Pj[m] = D1(pj[m], dir == 7 + m ? (T)1 : (T)0);
    }
    const D1 dD(d, dir == 14 ? (T)1 : (T)0);
    D1 rD[2], JD[2][13];
    edge_full<D1>(Pi, Pj, dD, D1(xh0, (T)0), D1(xh1, (T)0), D1(fx, (T)0), D1(fy, (T)0), D1(cx, (T)0),
                  D1(cy, (T)0), D1(z_min, (T)0), tx, ty, rD, JD);
    T acc = (T)0;
    for (int c = 0; c < 2; ++c) {
      acc += rb[c] * rD[c].d;
      for (int m = 0; m < 13; ++m) acc += Jb[c][m] * JD[c][m].d;
    }
    xb[dir] = acc;
  }
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
  hipLaunchKernelGGL((edge_adjoint_kernel<T>), dim3(blocks_for(4LL * n_edges, 256), n), dim3(256), 0, st, G, it);
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
