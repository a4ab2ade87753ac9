// Damped solve of a reduced camera system S dxi = s of moderate size (DPV-SLAM
// Appendix A: the Cholesky factorisation of the pose block of the Schur
// complement) by one workgroup, which factors S in LDS (packed lower
// triangle) and runs both triangular solves.  Larger systems take the
// block-sparse factor (sparse.hip).
//
// S is dense row-major n x n; only its lower triangle is read.  A pivot that
// is not positive (or not finite) sets *status and is replaced by 1 so the
// arithmetic stays finite; the step is then zero.  min_pivot receives the
// smallest L_ii^2 / S_ii (as ordered bits of a non-negative float, combined
// with an integer atomic minimum, which is order-independent).
#include <algorithm>

#include "common.h"
#include "packed.h"

namespace dpvba {

__device__ __forceinline__ void pivot_min(unsigned int* min_bits, float ratio) {
  if (!(ratio >= 0.f)) ratio = 0.f;
  atomicMin(min_bits, __float_as_uint(ratio));
}

constexpr int kSmallCholThreads = 512;
template <typename T>
__global__ void __launch_bounds__(kSmallCholThreads) small_chol_solve_kernel(const T* S, const T* rhs, int n, T* dx,
                                                               int* status, unsigned int* min_bits) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  T* d0 = reinterpret_cast<T*>(dyn_lds);  // [n] damped diagonal (pivot report)
  T* invd = d0 + n;                       // [n]
  T* piv = invd + n;                      // [n]
  T* x = piv + n;                         // [n]
  T* A = x + n;                           // packed lower, row i at i(i+1)/2; s appended as row n
  __shared__ int bad;
  __shared__ unsigned int minr_bits;
  const int tid = threadIdx.x;
  if (n + 1 <= kSmallRows) {  // the small panel solver
    __shared__ float minr;
    const int nr = small_solve_rows(n);
    T* xr = reinterpret_cast<T*>(dyn_lds) + small_solve_x(nr);  // after the solver's own arrays
    panel_chol_solve<T>(n, S, rhs, nullptr, dyn_lds, xr, &bad, &minr, n, [] {});
    for (int i = tid; i < n; i += blockDim.x) dx[i] = xr[i];  // zero when a pivot failed
    if (tid == 0) {
      if (bad) atomicOr(status, 1);
      pivot_min(min_bits, minr);
    }
    return;
  }
  const int np = n * (n + 1) / 2;
  // lower triangle of the dense row-major S, eight independent loads in
  // flight per thread
  const int nn = n * n;
  for (int q0 = tid; q0 < nn; q0 += 8 * blockDim.x) {
    T v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = q0 + u * blockDim.x, i = q / n, j = q - (q / n) * n;
      v[u] = (q < nn && j <= i) ? S[q] : (T)0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = q0 + u * blockDim.x, i = q / n, j = q - (q / n) * n;
      if (q < nn && j <= i) {
        A[packed_index(i, j)] = v[u];
        if (i == j) d0[i] = v[u];
      }
    }
  }
  for (int i = tid; i < n; i += blockDim.x) A[np + i] = rhs[i];
  if (tid == 0) {
    A[np + n] = (T)0;
    bad = 0;
    minr_bits = __float_as_uint(3.0e38f);
  }
  __syncthreads();
  packed_panel_factor<T>(A, n, n + 1, invd, piv, &bad);  // row n ends as y = L^-1 s
  pivot_ratio_min<T>(piv, d0, n, &minr_bits);              // smallest pivot / damped diagonal
  packed_back_solve<T>(A, n, invd, A + np, x);
  __syncthreads();
  for (int i = tid; i < n; i += blockDim.x) dx[i] = bad ? (T)0 : x[i];
  if (tid == 0) {
    if (bad) atomicOr(status, 1);
    pivot_min(min_bits, __uint_as_float(minr_bits));
  }
}

// packed panel factor in LDS; the substitutions keep the vector on one
// wavefront (n <= 255)
int small_solve_max_n(int tsize) { return tsize == 4 ? 240 : 160; }

// dx = S^-1 rhs for 0 < n <= small_solve_max_n.
template <typename T>
hipError_t launch_small_chol(const T* S, const T* rhs, int n, T* dx, int* status, unsigned int* min_bits,
                             hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (n > small_solve_max_n(sizeof(T))) return hipErrorInvalidValue;
  const int lds = n + 1 <= kSmallRows
                      ? std::max(packed_solve_lds_bytes(n, sizeof(T)), small_solve_lds_bytes(n, sizeof(T)))
                      : packed_solve_lds_bytes(n, sizeof(T));
  hipError_t e = opt_in_lds((const void*)small_chol_solve_kernel<T>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((small_chol_solve_kernel<T>), dim3(1), dim3(kSmallCholThreads), lds, st, S, rhs, n, dx, status, min_bits);
  return hipGetLastError();
}

template hipError_t launch_small_chol<float>(const float*, const float*, int, float*, int*, unsigned int*, hipStream_t);
template hipError_t launch_small_chol<double>(const double*, const double*, int, double*, int*, unsigned int*,
                                              hipStream_t);

}  // namespace dpvba
