// Mixed-precision solve of the reduced camera system (DPV-SLAM Appendix A:
// the Cholesky factorisation of the Schur complement's pose block, here in
// float32 on the matrix cores, with float64 iterative refinement).
//
// Given S64 (float64 block storage of an elimination plan) and s64 gathered from the float32 tile
// shares: factor S32 = fl32(S64) once, solve, then repeat
//   r = s64 - S64 x   (float64),   x += (L L^T)^-1 fl32(r)
// a fixed number of times (the last left out at a residual where it gains
// nothing; sparse.hip holds the steps).  The iteration is accepted when
// max |r| <= tol max |s64| after the last step; otherwise (or when the
// float32 factorisation met a non-positive pivot) the caller re-solves with
// a float64 Cholesky of S64.
#include "common.h"

namespace dpvba {

// Accept or fall back; records the relative residual and the decision.
__global__ void refine_decide_kernel(const unsigned long long* m, const int* status32, double tol, int force,
                                     double* resid_out, int* fallback_out, int* host_flag) {
  if (threadIdx.x != 0) return;
  const double rmax = __longlong_as_double((long long)m[0]);
  const double smax = __longlong_as_double((long long)m[1]);
  const double rel = smax > 0.0 ? rmax / smax : rmax;
  const int fb = force || (*status32 != 0) || !(rel <= tol);
  *resid_out = rel;
  *fallback_out = fb;
  *host_flag = fb;
}

// Final step in the state precision, from the plan's padded rows to the poses' order.  The iteration's status becomes that of
// the solve actually used: the float32 one when accepted (then clean), else
// the float64 fallback's; a failed fallback leaves a zero step.
__global__ void step_to_f32_kernel(const double* x, const int* row0, float* dx, int n, const int* fallback,
                                   const int* status64, int* status) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  const int fb = *fallback;
  const int bad = fb && *status64;
  if (q < n) dx[q] = bad ? 0.f : (float)x[row0[q / 6] + q % 6];
  if (q == 0) *status = fb ? *status64 : 0;
}

static inline unsigned nblocks(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_refine_decide(const unsigned long long* maxes, const int* status32, double tol, int force,
                                double* resid_out, int* fallback_out, int* host_flag, hipStream_t st) {
  hipLaunchKernelGGL(refine_decide_kernel, dim3(1), dim3(64), 0, st, maxes, status32, tol, force, resid_out,
                     fallback_out, host_flag);
  return hipGetLastError();
}

hipError_t launch_step_to_f32(const double* x, const int* row0, float* dx, int n, const int* fallback,
                              const int* status64, int* status, hipStream_t st) {
  hipLaunchKernelGGL(step_to_f32_kernel, dim3(nblocks(n > 0 ? n : 1, 256)), dim3(256), 0, st, x, row0, dx, n, fallback,
                     status64, status);
  return hipGetLastError();
}

}  // namespace dpvba
