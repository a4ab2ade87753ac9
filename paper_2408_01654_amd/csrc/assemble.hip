// Large-path and auxiliary kernels: gather of the tiles' shares into the
// dense damped reduced camera system (DPV-SLAM Appendix A), per-edge cost of
// eq. (3) at an iterate, report reductions, and the full-patch reprojection
// of eq. (2).
#include "edge.h"
#include "dpvba.h"

namespace dpvba {

// Gather of the per-tile vectors into the right-hand side s and Diag(B):
// one wavefront per free pose P, lane l summing the pose's shares l, l + 64,
// ... (six right-hand-side and six Diag(B) entries each), then a butterfly
// over the lanes; fixed order, so the result is reproducible.  The shares
// (type TP) are summed in the output type T, so float shares gathered into
// double are combined without further rounding error.  With row0, free pose
// P's rows start at row0[P] (an elimination plan's padded order; null: the
// poses' own order).
template <typename TP, typename T>
__global__ void __launch_bounds__(256) gather_vec_kernel(const TP* part_vec, const int* off, const int2* src,
                                                         int n_free, T* rhs, T* dB, const int* row0) {
  const int P_ = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (P_ >= n_free) return;
  T v[6], d[6];
#pragma unroll
  for (int m = 0; m < 6; ++m) v[m] = d[m] = (T)0;
  for (int q = off[P_] + lane; q < off[P_ + 1]; q += 64) {
    const int2 sq = src[q];
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      v[m] += (T)part_vec[sq.x + m];
      d[m] += (T)part_vec[sq.y + m];
    }
  }
#pragma unroll
  for (int h = 32; h >= 1; h >>= 1)
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      v[m] += __shfl_xor(v[m], h);
      d[m] += __shfl_xor(d[m], h);
    }
  if (lane < 6) {
    T vv = v[0], dd = d[0];
#pragma unroll
    for (int m = 1; m < 6; ++m)
      if (lane == m) {
        vv = v[m];
        dd = d[m];
      }
    const int xd = (row0 ? row0[P_] : 6 * P_) + lane;
    rhs[xd] = vv;
    dB[xd] = dd;
  }
}

// Gather of every lower 6x6 block (P >= Q) of the damped reduced system from
// the tile partials (zero where no tile contributes), with the damping
// lam_diag Diag(B) + lambda added to the diagonal.  `mirror` also writes the
// upper triangle.
template <typename TP, typename T>
__global__ void gather_S_kernel(const TP* part_S, const int* off, const int* src, int n_free, T* S,
                                const T* dB, T lambda, T lam_diag, int mirror, T* diag_out) {
  const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nblk = (long long)n_free * (n_free + 1) / 2;
  if (g >= nblk * 36) return;
  const int blk = (int)(g / 36), e = (int)(g % 36), r = e / 6, c = e % 6;
  int Pb, Qb;
  lower_block_of(blk, Pb, Qb);
  if (Pb == Qb && r < c) return;
  T v = (T)0;
  const int lo = off[blk], hi = off[blk + 1];
  const int eo = c * 6 + r;  // the tiles store upper entries of their block pairs
  int q = lo;
  for (; q + 4 <= hi; q += 4) {
    const T v0 = (T)part_S[src[q] + eo], v1 = (T)part_S[src[q + 1] + eo];
    const T v2 = (T)part_S[src[q + 2] + eo], v3 = (T)part_S[src[q + 3] + eo];
    v += v0; v += v1; v += v2; v += v3;
  }
  for (; q < hi; ++q) v += (T)part_S[src[q] + eo];
  const int n = 6 * n_free;
  const int row = 6 * Pb + r, col = 6 * Qb + c;
  if (row == col) {
    v += lam_diag * dB[row] + lambda;
    if (diag_out) diag_out[row] = v;
  }
  S[(size_t)row * n + col] = v;
  if (mirror && row != col) S[(size_t)col * n + row] = v;
}

// Cost of every edge at an iterate, summed per block in a fixed order.
template <typename T, typename P>
__global__ void __launch_bounds__(256) edge_cost_kernel(const P* poses, const P* inv_depth,
                                                         const float* patches, int p, const int* ii,
                                                         const int* jj, const int* kk,
                                                         const float* target, const float* weight,
                                                         int n_edges, T fx, T fy, T cx, T cy, T z_min,
                                                         double* part) {
  __shared__ double sred[256];
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  double cst = 0.0;
  if (e < n_edges) {
    T Ri[9], Rj[9], ti_[3], tj[3], Rt[12];
    const P* pi = poses + 7 * (size_t)ii[e];
    const P* pj = poses + 7 * (size_t)jj[e];
    quat_to_rot<T, P>(pi + 3, Ri);
    quat_to_rot<T, P>(pj + 3, Rj);
    for (int m = 0; m < 3; ++m) { ti_[m] = (T)pi[m]; tj[m] = (T)pj[m]; }
    relative_pose<T>(Ri, ti_, Rj, tj, Rt, Rt + 9);
    const int k = kk[e], c = (p - 1) / 2;
    const float* cen = patches + ((size_t)k * p * p + (size_t)c * p + c) * 2;
    EdgeTerms<T> o;
    const float2 tg = reinterpret_cast<const float2*>(target)[e];
    const float2 wt = reinterpret_cast<const float2*>(weight)[e];
    if (edge_eval<T>(Rt, ((T)cen[0] - cx) / fx, ((T)cen[1] - cy) / fy, (T)inv_depth[k], fx, fy, cx,
                     cy, z_min, tg.x, tg.y, wt.x, wt.y, o))
      cst = 0.5 * ((double)o.w[0] * o.r[0] * o.r[0] + (double)o.w[1] * o.r[1] * o.r[1]);
  }
  sred[threadIdx.x] = cst;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) sred[threadIdx.x] += sred[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sred[0];
}

// Reduce per-tile costs / invalid counts of one iteration into the report.
__global__ void report_reduce_kernel(const double* part_cost, const int* part_invalid, int n,
                                     double* cost_out, int* invalid_out) {
  __shared__ double sc[256];
  __shared__ int si[256];
  double c = 0.0;
  int v = 0;
  // fixed partition: thread t sums a contiguous range, then a fixed tree
  const int per = (n + 255) / 256;
  const int lo = threadIdx.x * per, hi = min(n, lo + per);
  for (int q = lo; q < hi; ++q) {
    c += part_cost[q];
    if (part_invalid) v += part_invalid[q];
  }
  sc[threadIdx.x] = c;
  si[threadIdx.x] = v;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      sc[threadIdx.x] += sc[threadIdx.x + w];
      si[threadIdx.x] += si[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *cost_out = sc[0];
    if (invalid_out) *invalid_out = si[0];
  }
}

// Reprojection of every pixel of every edge's patch (eq. 2).  The output
// (8 p^2 bytes an edge) is most of the traffic, so a workgroup takes 256
// consecutive edges in two steps: thread e forms edge e's relative pose and
// inverse depth in LDS, then the threads walk the edges' pixels in output
// order, one pixel a thread, so that a wavefront writes 512 contiguous bytes
// (one thread per edge wrote 8 bytes every 8 p^2).  P2: the pixels of a patch
// when known at compile time (0: p * p), for the division of the walk.
// 1,505,568 edges of 3 x 3 patches: 127 us before, 47 us now (2.7 TB/s of the
// 125 MB it has to move).
constexpr int kReprojLd = 13;  // R (9), t d (3), inverse depth d; odd, so neighbouring edges lie on different banks

template <typename T, int P2>
__global__ void __launch_bounds__(256) reproject_kernel(const float* poses, const float* inv_depth,
                                                        const float* patches, int p, const int* ii, const int* jj,
                                                        const int* kk, int n_edges, T fx, T fy, T cx, T cy, T z_min,
                                                        float* coords, uint8_t* valid) {
  __shared__ T sT[256 * kReprojLd];
  __shared__ int sK[256];
  const int e0 = blockIdx.x * 256;
  const int ne = min(256, n_edges - e0);
  const int p2 = P2 ? P2 : p * p;
  if ((int)threadIdx.x < ne) {
    const int e = e0 + threadIdx.x;
    T Ri[9], Rj[9], ti_[3], tj[3], R[9], t[3];
    const float* pi = poses + 7 * (size_t)ii[e];
    const float* pj = poses + 7 * (size_t)jj[e];
    quat_to_rot<T, float>(pi + 3, Ri);
    quat_to_rot<T, float>(pj + 3, Rj);
    for (int m = 0; m < 3; ++m) { ti_[m] = pi[m]; tj[m] = pj[m]; }
    relative_pose<T>(Ri, ti_, Rj, tj, R, t);
    T* o = sT + kReprojLd * threadIdx.x;
    for (int m = 0; m < 9; ++m) o[m] = R[m];
    const T d = inv_depth[kk[e]];
    for (int m = 0; m < 3; ++m) o[9 + m] = t[m] * d;
    o[12] = d;
    sK[threadIdx.x] = kk[e];
  }
  __syncthreads();
  const int c = (p - 1) / 2;
  float* out = coords + (size_t)e0 * p2 * 2;
  for (int x = threadIdx.x; x < ne * p2; x += 256) {
    const int le = x / p2, px = x - le * p2;
    const T* R = sT + kReprojLd * le;
    const T* td = R + 9;
    const T d = R[12];
    const float* pk = patches + ((size_t)sK[le] * p2 + px) * 2;
    const T u = ((T)pk[0] - cx) / fx, v = ((T)pk[1] - cy) / fy;
    const T q0 = R[0] * u + R[1] * v + R[2] + td[0];
    const T q1 = R[3] * u + R[4] * v + R[5] + td[1];
    const T q2 = R[6] * u + R[7] * v + R[8] + td[2];
    out[2 * x] = (float)(fx * q0 / q2 + cx);
    out[2 * x + 1] = (float)(fy * q1 / q2 + cy);
    if (valid && px == c * p + c) valid[e0 + le] = (d > (T)0 && q2 > z_min * d) ? 1 : 0;
  }
}

// Per-solve report state: step status words and pivot minima per iteration.
__global__ void report_init_kernel(int* status, unsigned int* min_bits, int n, int* err_clear) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    status[i] = 0;
    min_bits[i] = 0x7f7fffffu;  // bits of FLT_MAX
  }
  if (i == 0 && err_clear) *err_clear = 0;
}

__global__ void report_finalize_kernel(dpvba_report* rep, const int* status, const unsigned int* min_bits,
                                       int n_iters, const int* err, const double* refine, const int* fallback) {
  if (threadIdx.x != 0) return;
  int st = DPVBA_OK;
  for (int t = 0; t < n_iters; ++t) {
    if (status[t]) st = DPVBA_ENOTPD;
    rep->min_pivot[t] = (double)__uint_as_float(min_bits[t]);
    rep->refine_resid[t] = refine ? refine[t] : 0.0;
    rep->fp64_fallback[t] = fallback ? fallback[t] : 0;
  }
  if (err && (*err & kErrInput)) st = DPVBA_EINVAL;
  if (err && (*err & (kErrBarrier | kErrChain))) st = DPVBA_EHIP;
  rep->status = st;
  rep->n_iters = n_iters;
}

hipError_t launch_report_init(int* status, unsigned int* min_bits, int n, hipStream_t st, int* err_clear) {
  hipLaunchKernelGGL(report_init_kernel, dim3((n + 63) / 64), dim3(64), 0, st, status, min_bits, n, err_clear);
  return hipGetLastError();
}

hipError_t launch_report_finalize(dpvba_report* rep, const int* status, const unsigned int* min_bits,
                                  int n_iters, const int* err, hipStream_t st, const double* refine,
                                  const int* fallback) {
  hipLaunchKernelGGL(report_finalize_kernel, dim3(1), dim3(64), 0, st, rep, status, min_bits, n_iters, err, refine,
                     fallback);
  return hipGetLastError();
}

// ---------------------------------------------------------------- launchers

// rhs and Diag(B) alone, at the rows of an elimination plan.
template <typename TP, typename T>
hipError_t launch_gather_vec(const TP* part_vec, const int* v_off, const int2* v_src, int n_free, T* rhs, T* dB,
                             const int* row0, hipStream_t st) {
  if (n_free == 0) return hipSuccess;
  hipLaunchKernelGGL((gather_vec_kernel<TP, T>), dim3((n_free + 3) / 4), dim3(256), 0, st, part_vec, v_off, v_src,
                     n_free, rhs, dB, row0);
  return hipGetLastError();
}

template <typename TP, typename T>
hipError_t launch_gather_as(const TP* part_S, const TP* part_vec, const int* s_off, const int* s_src,
                            const int* v_off, const int2* v_src, int n_free, T* S, T* rhs, T* dB, T lambda,
                            T lam_diag, int mirror, T* diag_out, hipStream_t st) {
  if (n_free == 0) return hipSuccess;
  hipError_t e = launch_gather_vec<TP, T>(part_vec, v_off, v_src, n_free, rhs, dB, nullptr, st);
  if (e != hipSuccess) return e;
  const long long tot = (long long)n_free * (n_free + 1) / 2 * 36;
  hipLaunchKernelGGL((gather_S_kernel<TP, T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, part_S,
                     s_off, s_src, n_free, S, dB, lambda, lam_diag, mirror, diag_out);
  return hipGetLastError();
}

template <typename T, typename P>
hipError_t launch_edge_cost(const P* poses, const P* inv_depth, const float* patches, int p, const int* ii,
                            const int* jj, const int* kk, const float* target, const float* weight,
                            int n_edges, T fx, T fy, T cx, T cy, T z_min, double* part, hipStream_t st) {
  const int nblk = (n_edges + 255) / 256;
  if (nblk == 0) return hipSuccess;
  hipLaunchKernelGGL((edge_cost_kernel<T, P>), dim3(nblk), dim3(256), 0, st, poses, inv_depth, patches, p,
                     ii, jj, kk, target, weight, n_edges, fx, fy, cx, cy, z_min, part);
  return hipGetLastError();
}

hipError_t launch_report_reduce(const double* part_cost, const int* part_invalid, int n, double* cost_out,
                                int* invalid_out, hipStream_t st) {
  hipLaunchKernelGGL(report_reduce_kernel, dim3(1), dim3(256), 0, st, part_cost, part_invalid, n, cost_out,
                     invalid_out);
  return hipGetLastError();
}

hipError_t launch_reproject(const float* poses, const float* inv_depth, const float* patches, int p,
                            const int* ii, const int* jj, const int* kk, int n_edges, float fx, float fy,
                            float cx, float cy, float z_min, float* coords, uint8_t* valid, hipStream_t st) {
  if (n_edges == 0) return hipSuccess;
  // 3 x 3 patches (the odometry's): the walk's division is by a constant
  if (p == 3)
    hipLaunchKernelGGL((reproject_kernel<float, 9>), dim3((n_edges + 255) / 256), dim3(256), 0, st, poses, inv_depth,
                       patches, p, ii, jj, kk, n_edges, fx, fy, cx, cy, z_min, coords, valid);
  else
    hipLaunchKernelGGL((reproject_kernel<float, 0>), dim3((n_edges + 255) / 256), dim3(256), 0, st, poses, inv_depth,
                       patches, p, ii, jj, kk, n_edges, fx, fy, cx, cy, z_min, coords, valid);
  return hipGetLastError();
}

#define DPVBA_INSTANTIATE(T, P)                                                                        \
  template hipError_t launch_edge_cost<T, P>(const P*, const P*, const float*, int, const int*,        \
                                             const int*, const int*, const float*, const float*, int,  \
                                             T, T, T, T, T, double*, hipStream_t);

DPVBA_INSTANTIATE(float, float)
DPVBA_INSTANTIATE(double, double)
#define DPVBA_GATHER_INSTANTIATE(TP, T)                                                                              \
  template hipError_t launch_gather_vec<TP, T>(const TP*, const int*, const int2*, int, T*, T*, const int*,           \
                                               hipStream_t);                                                         \
  template hipError_t launch_gather_as<TP, T>(const TP*, const TP*, const int*, const int*, const int*, const int2*, \
                                              int, T*, T*, T*, T, T, int, T*, hipStream_t);
DPVBA_GATHER_INSTANTIATE(float, float)
DPVBA_GATHER_INSTANTIATE(double, double)
DPVBA_GATHER_INSTANTIATE(float, double)

}  // namespace dpvba
