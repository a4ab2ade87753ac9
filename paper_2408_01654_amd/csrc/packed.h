// Dense Cholesky factorisation and solves of one small symmetric system held
// as a packed lower triangle (row i at i (i + 1) / 2), by one workgroup.
// The storage may be shared memory or global memory private to the
// workgroup; every thread of the workgroup calls these functions.
#pragma once

#include "common.h"
#include "mfma.h"

namespace dpvba {

// 1 / sqrt(d) of a positive pivot: the hardware reciprocal square root for
// float32 (within about one unit in the last place, far inside the float32
// path's tolerance; it keeps the per-column dependency chain short); for float64 one
// third-order step on the hardware's estimate, within about one unit in the
// last place like 1 / sqrt(d), whose division and root are two long chains.
template <typename T>
__device__ __forceinline__ T pivot_rsqrt(T d) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_amdgcn_rsqf(d);
  } else {
    // y (1 + e / 2 + 3 e^2 / 8), e = 1 - d y^2: the third-order step leaves
    // e^3, far below the last bit
    const T y = __builtin_amdgcn_rsq(d);
    const T e = __builtin_fma(-d * y, y, (T)1);
    return __builtin_fma(y * e, __builtin_fma(e, (T)0.375, (T)0.5), y);
  }
}

// Smallest pivot / damped-diagonal ratio of columns 0..n-1 (the bits of a
// non-negative float, a NaN counting as 0) combined into *min_bits: every
// thread takes columns tid, tid + blockDim.x, ..., each wavefront reduces its
// lanes with shuffles, and one lane per wavefront issues the atomic minimum
// (one LDS atomic per wavefront instead of one per column).  Called by every
// thread of the workgroup.
template <typename T>
__device__ __forceinline__ void pivot_ratio_min(const T* piv, const T* dd, int n, unsigned int* min_bits,
                                                int first = -1, int stride = 0) {
  unsigned int m = __float_as_uint(3.0e38f);
  if (first < 0) {
    first = threadIdx.x;
    stride = blockDim.x;
  }
  for (int j = first; j < n; j += stride) {
    const float ratio = (float)(piv[j] / dd[j]);
    m = min(m, __float_as_uint(ratio == ratio ? fmaxf(ratio, 0.f) : 0.f));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = min(m, (unsigned int)__shfl_xor((int)m, o));
  if ((threadIdx.x & 63) == 0) atomicMin(min_bits, m);
}

__device__ __forceinline__ int packed_index(int i, int j) { return i * (i + 1) / 2 + j; }

// In-place A = L L^T, right-looking with the column scaling deferred: step j
// subtracts A_ij A_kj / d_j from the trailing entries (j < k <= i), where
// d_j = A_jj after the earlier steps, so one barrier per column suffices;
// a final pass scales column j by 1 / sqrt(d_j).  The trailing entries are
// spread over a 16 x 16 thread grid (entry (i, k) on the thread with
// i = ty, k = tx mod 16), which needs blockDim.x >= 256 (threads beyond 256
// idle).  A pivot that is not positive or not finite is replaced by 1 and
// counted in *bad; *minr receives the smallest pivot / d0 ratio.  bad and
// minr live in shared memory.
template <typename TA>
__device__ __forceinline__ TA packed_pivot(TA d) {
  return (d > (TA)0 && d < (TA)3.0e38) ? d : (TA)1;
}

template <typename TA>
__device__ void packed_cholesky(TA* A, int n, const TA* d0, int* bad, float* minr) {
  const int tid = threadIdx.x;
  const int ty = tid & 15, tx = (tid >> 4) & 15;
  const bool worker = tid < 256;
  if (tid == 0) { *bad = 0; *minr = 3.0e38f; }
  __syncthreads();
  const int nb = (n + 15) >> 4;
  for (int j = 0; j < n; ++j) {
    const TA dj = A[packed_index(j, j)];
    if (tid == 0) {
      const float ratio = (float)(dj / d0[j]);
      if (ratio < *minr || !(ratio == ratio)) *minr = ratio == ratio ? ratio : 0.f;
      if (!(dj > (TA)0) || !(dj < (TA)3.0e38)) *bad = 1;
    }
    const TA inv = (TA)1 / packed_pivot(dj);
    if (worker) {
      for (int bi = (j + 1) >> 4; bi < nb; ++bi) {
        const int i = 16 * bi + ty;
        if (i <= j || i >= n) continue;
        const TA aij = A[packed_index(i, j)] * inv;
        TA* row = A + packed_index(i, 0);
        for (int bk = (j + 1) >> 4; bk <= bi; ++bk) {
          const int k = 16 * bk + tx;
          if (k > j && k <= i) row[k] -= aij * A[packed_index(k, j)];
        }
      }
    }
    __syncthreads();
  }
  // L_ij = A_ij / sqrt(d_j) (i > j), L_jj = sqrt(d_j)
  for (int i = tid; i < n; i += blockDim.x) {
    TA* row = A + packed_index(i, 0);
    for (int j = 0; j < i; ++j) row[j] /= dsqrt(packed_pivot(A[packed_index(j, j)]));
  }
  __syncthreads();
  for (int j = tid; j < n; j += blockDim.x) A[packed_index(j, j)] = dsqrt(packed_pivot(A[packed_index(j, j)]));
  __syncthreads();
}

// b <- (L L^T)^-1 b in place (n <= 256): both substitutions run in the
// first wavefront with b held in registers (row i on lane i mod 64) and
// each solved entry broadcast by a lane shuffle; no workgroup barrier inside.
template <typename TA, typename TB>
__device__ void packed_solve(const TA* L, TB* b, int n) {
  const int lane = threadIdx.x;
  if (lane < 64) {
    TB r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = (lane + 64 * q < n) ? b[lane + 64 * q] : (TB)0;
    // forward: L y = b
    for (int j = 0; j < n; ++j) {
      const int qj = j >> 6;
      TB bj = (TB)0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q == qj) bj = r[q];
      const TB yj = __shfl(bj, j & 63) / (TB)L[packed_index(j, j)];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = lane + 64 * q;
        if (i == j) r[q] = yj;
        else if (i > j && i < n) r[q] -= (TB)L[packed_index(i, j)] * yj;
      }
    }
    // backward: L^T x = y
    for (int j = n - 1; j >= 0; --j) {
      const int qj = j >> 6;
      TB yj = (TB)0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q == qj) yj = r[q];
      const TB xj = __shfl(yj, j & 63) / (TB)L[packed_index(j, j)];
      const TA* rowj = L + packed_index(j, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = lane + 64 * q;
        if (i == j) r[q] = xj;
        else if (i < j) r[q] -= (TB)rowj[i] * xj;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (lane + 64 * q < n) b[lane + 64 * q] = r[q];
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Packed systems of up to 255 unknowns on one workgroup of 256 threads or
// more: blocked factor and wavefront substitutions.

// Value of v on lane c of each 16-lane row, for every lane of that row
// (the DPP row broadcast of CDNA; c must fold to a constant).  The result
// stays in a vector register: no scalar register, no readlane hazard.
template <int C>
__device__ __forceinline__ int row_bcast_bits(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + C, 0xF, 0xF, true);
}
__device__ __forceinline__ int row_bcast_i(int v, int c) {
  switch (c) {
    case 0: return row_bcast_bits<0>(v);
    case 1: return row_bcast_bits<1>(v);
    case 2: return row_bcast_bits<2>(v);
    case 3: return row_bcast_bits<3>(v);
    case 4: return row_bcast_bits<4>(v);
    case 5: return row_bcast_bits<5>(v);
    case 6: return row_bcast_bits<6>(v);
    case 7: return row_bcast_bits<7>(v);
    case 8: return row_bcast_bits<8>(v);
    case 9: return row_bcast_bits<9>(v);
    case 10: return row_bcast_bits<10>(v);
    case 11: return row_bcast_bits<11>(v);
    case 12: return row_bcast_bits<12>(v);
    case 13: return row_bcast_bits<13>(v);
    case 14: return row_bcast_bits<14>(v);
    default: return row_bcast_bits<15>(v);
  }
}
template <typename T>
__device__ __forceinline__ T row_bcast(T v, int c) {
  if constexpr (sizeof(T) == 4) {
    return __int_as_float(row_bcast_i(__float_as_int(v), c));
  } else {
    const long long bits = __double_as_longlong(v);
    const int lo = row_bcast_i((int)(bits & 0xffffffffLL), c);
    const int hi = row_bcast_i((int)(bits >> 32), c);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
  }
}

// acc -= x * (x of the row's lane C): row_newbcast inside the multiply-add, so
// that a broadcast costs no instruction of its own (a separate move per
// column entry is a third of a float32 panel's instructions, half of a
// float64 one's).  Each statement opens with the two wait states a lane
// broadcast needs after the write of x, which the compiler cannot see in here.
// ROW_FMAC_n: columns C .. C + n - 1 of two rows a, b (na = -x_a, nb = -x_b).
template <typename T> struct RowFmac;
template <> struct RowFmac<float> {
  // column C of both rows, then the row's entry (C, C) to every lane
  template <int C>
  static __device__ __forceinline__ float next(float* a, float* b, float x, float na, float nb) {
    float d;
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %1, %3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 0\n\t"
                 "v_mov_b32_dpp %2, %0 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C]), "+&v"(b[C]), "=&v"(d)
                 : "v"(x), "v"(na), "v"(nb), "n"(C));
    return d;
  }
  template <int C>
  static __device__ __forceinline__ void cols1(float* a, float* b, float x, float na, float nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %1, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0));
  }
  template <int C>
  static __device__ __forceinline__ void cols2(float* a, float* b, float x, float na, float nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %1, %4, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %3, %4, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0]), "+&v"(a[C + 1]), "+&v"(b[C + 1])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0), "n"(C + 1));
  }
  template <int C>
  static __device__ __forceinline__ void cols4(float* a, float* b, float x, float na, float nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %8, %9 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %1, %8, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %2, %8, %9 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %3, %8, %10 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %4, %8, %9 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %5, %8, %10 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %6, %8, %9 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %7, %8, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0]), "+&v"(a[C + 1]), "+&v"(b[C + 1]), "+&v"(a[C + 2]), "+&v"(b[C + 2]), "+&v"(a[C + 3]), "+&v"(b[C + 3])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0), "n"(C + 1), "n"(C + 2), "n"(C + 3));
  }
  template <int C>
  static __device__ __forceinline__ void cols6(float* a, float* b, float x, float na, float nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f32_dpp %0, %12, %13 row_newbcast:%15 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %1, %12, %14 row_newbcast:%15 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %2, %12, %13 row_newbcast:%16 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %3, %12, %14 row_newbcast:%16 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %4, %12, %13 row_newbcast:%17 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %5, %12, %14 row_newbcast:%17 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %6, %12, %13 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %7, %12, %14 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %8, %12, %13 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %9, %12, %14 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %10, %12, %13 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f32_dpp %11, %12, %14 row_newbcast:%20 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0]), "+&v"(a[C + 1]), "+&v"(b[C + 1]), "+&v"(a[C + 2]), "+&v"(b[C + 2]), "+&v"(a[C + 3]), "+&v"(b[C + 3]), "+&v"(a[C + 4]), "+&v"(b[C + 4]), "+&v"(a[C + 5]), "+&v"(b[C + 5])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0), "n"(C + 1), "n"(C + 2), "n"(C + 3), "n"(C + 4), "n"(C + 5));
  }
};

template <> struct RowFmac<double> {
  // column C of both rows, then the row's entry (C, C) to every lane
  template <int C>
  static __device__ __forceinline__ double next(double* a, double* b, double x, double na, double nb) {
    double d;
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 0\n\t"
                 "v_mov_b64_dpp %2, %0 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C]), "+&v"(b[C]), "=&v"(d)
                 : "v"(x), "v"(na), "v"(nb), "n"(C));
    return d;
  }
  template <int C>
  static __device__ __forceinline__ void cols1(double* a, double* b, double x, double na, double nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0));
  }
  template <int C>
  static __device__ __forceinline__ void cols2(double* a, double* b, double x, double na, double nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %4, %6 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %3, %4, %6 row_newbcast:%8 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0]), "+&v"(a[C + 1]), "+&v"(b[C + 1])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0), "n"(C + 1));
  }
  template <int C>
  static __device__ __forceinline__ void cols4(double* a, double* b, double x, double na, double nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %8, %9 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %8, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %2, %8, %9 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %3, %8, %10 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %4, %8, %9 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %5, %8, %10 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %6, %8, %9 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %7, %8, %10 row_newbcast:%14 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0]), "+&v"(a[C + 1]), "+&v"(b[C + 1]), "+&v"(a[C + 2]), "+&v"(b[C + 2]), "+&v"(a[C + 3]), "+&v"(b[C + 3])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0), "n"(C + 1), "n"(C + 2), "n"(C + 3));
  }
  template <int C>
  static __device__ __forceinline__ void cols6(double* a, double* b, double x, double na, double nb) {
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %12, %13 row_newbcast:%15 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %12, %14 row_newbcast:%15 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %2, %12, %13 row_newbcast:%16 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %3, %12, %14 row_newbcast:%16 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %4, %12, %13 row_newbcast:%17 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %5, %12, %14 row_newbcast:%17 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %6, %12, %13 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %7, %12, %14 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %8, %12, %13 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %9, %12, %14 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %10, %12, %13 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %11, %12, %14 row_newbcast:%20 row_mask:0xf bank_mask:0xf"
                 : "+&v"(a[C + 0]), "+&v"(b[C + 0]), "+&v"(a[C + 1]), "+&v"(b[C + 1]), "+&v"(a[C + 2]), "+&v"(b[C + 2]), "+&v"(a[C + 3]), "+&v"(b[C + 3]), "+&v"(a[C + 4]), "+&v"(b[C + 4]), "+&v"(a[C + 5]), "+&v"(b[C + 5])
                 : "v"(x), "v"(na), "v"(nb), "n"(C + 0), "n"(C + 1), "n"(C + 2), "n"(C + 3), "n"(C + 4), "n"(C + 5));
  }
};

// Columns C .. 15.
template <typename T, int C>
__device__ __forceinline__ void row_fmac_rest(T* a, T* b, T x, T na, T nb) {
  if constexpr (C + 6 <= 16) {
    RowFmac<T>::template cols6<C>(a, b, x, na, nb);
    row_fmac_rest<T, C + 6>(a, b, x, na, nb);
  } else if constexpr (C + 4 <= 16) {
    RowFmac<T>::template cols4<C>(a, b, x, na, nb);
    row_fmac_rest<T, C + 4>(a, b, x, na, nb);
  } else if constexpr (C + 2 <= 16) {
    RowFmac<T>::template cols2<C>(a, b, x, na, nb);
    row_fmac_rest<T, C + 2>(a, b, x, na, nb);
  } else if constexpr (C < 16) {
    RowFmac<T>::template cols1<C>(a, b, x, na, nb);
  }
}

// Whether a reciprocal square root is that of a positive finite pivot.
__device__ __forceinline__ bool good_rsqrt(float rs) { return __builtin_amdgcn_classf(rs, 0x180); }
__device__ __forceinline__ bool good_rsqrt(double rs) { return __builtin_amdgcn_class(rs, 0x180); }

// Cholesky of 16 columns on one wavefront, rows in registers: every 16-lane
// row of the wavefront holds the 16 x 16 diagonal block in a (lane s: row s),
// each lane one row below it in b.  Column c: scale it, update column c + 1
// and start that column's pivot at once, so that the chain of pivots runs
// beside the other columns' updates.  A pivot that is not positive and
// finite sets bad and leaves its column unscaled.  Entries above the diagonal are never
// read as results.
template <typename T, int C = 0>
__device__ __forceinline__ void chol16_columns(T* a, T* b, T rs, int& bad) {
  const bool ok = good_rsqrt(rs);
  bad |= !ok;
  rs = ok ? rs : (T)1;
  a[C] *= rs;
  b[C] *= rs;
  if constexpr (C < 15) {
    const T x = a[C], na = -a[C], nb = -b[C];
    const T d = RowFmac<T>::template next<C + 1>(a, b, x, na, nb);
    const T rn = pivot_rsqrt<T>(d);
    __builtin_amdgcn_sched_barrier(0);  // the estimate is under way before the other columns
    row_fmac_rest<T, C + 2>(a, b, x, na, nb);
    chol16_columns<T, C + 1>(a, b, rn, bad);
  }
}

template <typename T>
__device__ __forceinline__ void chol16(T* a, T* b, int& bad) {
  chol16_columns<T>(a, b, pivot_rsqrt<T>(row_bcast(a[0], 0)), bad);
}

// Value of v on lane l (uniform) of the wavefront.
template <typename T>
__device__ __forceinline__ T lane_bcast(T v, int l) {
  if constexpr (sizeof(T) == 4) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
  } else {
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(bits & 0xffffffffLL), l);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
  }
}

// Rank-16 update of a small system's matrix by panel p: the 16 x 16 blocks
// (bi, bk), bk = bk_lo .. bk_hi, bi = bk .. mb (the right-hand side's block),
// go to the wavefronts first, first + nwav, ...: W_(bi,bk) -= W_(bi,p) W_(bk,p)^T.
template <typename T>
__device__ __forceinline__ void panel_update(T* W, int ldw, int mb, int p, int bk_lo, int bk_hi, int first, int nwav) {
  const int lane = threadIdx.x & 63, c0 = 16 * p;
  int bk = bk_lo, bi = bk + first;
#pragma unroll 1
  for (;;) {
    while (bk <= bk_hi && bi > mb) {  // past this column block: on into the next
      bi += bk - mb;
      ++bk;
    }
    if (bk > bk_hi) break;
    const T* xr = W + (16 * bi + (lane & 15)) * ldw + c0 + (lane >> 4);
    const T* yr = W + (16 * bk + (lane & 15)) * ldw + c0 + (lane >> 4);
    T* out = W + 16 * bi * ldw + 16 * bk + (lane & 15);
    T old[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) old[v] = out[Mfma<T>::row(lane, v) * ldw];
    typename Mfma<T>::acc_t acc = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 16; k += 4) acc = Mfma<T>::step(xr[k], yr[k], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) out[Mfma<T>::row(lane, v) * ldw] = old[v] - acc[v];
    bi += nwav;
  }
}

// Cholesky solve S x = s of a small system (n <= 95) by one workgroup of at
// least four wavefronts: the matrix in LDS, padded to mb 16-column panels with
// an identity, the right-hand side as row block mb (its first row, which ends
// as y = L^-1 s; its other rows are never looked at).  Panel p: each of the
// first one or two wavefronts factors the 16 x 16 diagonal block and takes four
// of the row blocks below it (chol16), while the others finish the update
// by panel p - 1 on the matrix cores; after one barrier everyone updates the
// next column block, and a second closes the panel.  The factored diagonal
// blocks are kept apart, since the second wavefront may still read the block.
// Then L^T x = y on wavefront 0, the pivot report on wavefront 1, and
// beside() on all but the first.  The loops over panels are rolled: the code
// runs once or twice a launch, and with the matrix in registers and everything
// unrolled most of the time went into fetching instructions (factor, solve and
// retraction of 90 float64 unknowns in a launch of their own: 31.4 -> 22.8 us; a
// 22-frame window of two iterations in float32: 153.4 -> 124.2 us).
// x [n] (LDS): zero if a pivot was not positive.  ld > 0: Sp_g is a dense
// row-major matrix with row stride ld (its lower triangle is read), else
// packed; d0_g null: the damped diagonal is that of S.  The arrays fit the
// small_solve_x(nr) entries before x (nr = small_solve_rows(n)).
template <typename T, typename F>
__device__ __forceinline__ void panel_chol_solve(int n_in, const T* Sp_g, const T* rhs_g, const T* d0_g,
                                                 unsigned char* lds, T* x, int* bad_out, float* minr_out, int ld,
                                                 F&& beside) {
  constexpr int kDs = 16 * 17;
  const int n = __builtin_amdgcn_readfirstlane(n_in);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nwav = (int)blockDim.x >> 6;
  // rows on 16 bytes, and 16-row operand reads on different banks
  const int mb = (n + 15) >> 4, nrp = 16 * mb, ldw = nrp + 16 / (int)sizeof(T);
  T* W = reinterpret_cast<T*>(lds);  // [nrp + 16][ldw]
  T* Ld = W + (nrp + 16) * ldw;      // [mb][16][17] factored diagonal blocks
  T* dd = Ld + mb * kDs;             // [nrp] damped diagonal
  for (int k = tid; k < nrp; k += blockDim.x) {
    W[nrp * ldw + k] = k < n ? rhs_g[k] : (T)0;
    if (d0_g && k < n) dd[k] = d0_g[k];
  }
  {
    const int ty = (tid >> 4) & 15, tx = tid & 15, parts = (int)blockDim.x >> 8;
    const int nt = mb * (mb + 1) / 2;
    for (int t0 = w >> 2; t0 < nt; t0 += 8 * parts) {  // eight 16 x 16 tiles' loads in flight
      T v[8];
      int at[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = min(t0 + u * parts, nt - 1);
        int bi = 0;
        while ((bi + 1) * (bi + 2) / 2 <= t) ++bi;
        const int i = 16 * bi + ty, k = 16 * (t - bi * (bi + 1) / 2) + tx;
        at[u] = i * ldw + k;
        if (i < n && k <= i) v[u] = ld > 0 ? Sp_g[(size_t)i * ld + k] : Sp_g[i * (i + 1) / 2 + k];
        else v[u] = (T)(i == k ? 1 : 0);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) W[at[u]] = v[u];
    }
  }
  __syncthreads();
  if (!d0_g) {
    if (tid < n) dd[tid] = W[tid * ldw + tid];
    __syncthreads();
  }
  int bad = 0;
#pragma unroll 1
  for (int p = 0; p < mb; ++p) {
    const int act = mb - p > 4 ? 2 : 1;  // wavefronts on the panel
    if (w < act) {
      const int s = lane & 15, q = lane >> 4, bq = p + 1 + 4 * w + q;
      const T* wa = W + (16 * p + s) * ldw + 16 * p;
      T* wb = W + (bq <= mb ? 16 * bq + s : nrp + 15) * ldw + 16 * p;  // else a row nobody looks at
      T ra[16], rb[16];
      get_row<T, 16>(wa, ra);
      get_row<T, 16>(wb, rb);
      chol16<T>(ra, rb, bad);
      // (the stores that depend on the lane come last: a branch here would sink
      // the rows' updates below it)
      put_row<T, 16>(wb, rb);
      if (lane < 16 && w == 0) {
#pragma unroll
        for (int c = 0; c < 16; ++c) Ld[p * kDs + s * 17 + c] = ra[c];
      }
    } else if (p > 0) {
      panel_update<T>(W, ldw, mb, p - 1, p + 1, mb - 1, w - act, nwav - act);
    }
    __syncthreads();
    if (p + 1 < mb) panel_update<T>(W, ldw, mb, p, p + 1, p + 1, w, nwav);
    __syncthreads();
  }
  if (w == 0) {  // backward substitution; lane l holds entries l, l + 64
    const int r0 = lane, r1 = lane + 64;
    T y0 = r0 < n ? W[nrp * ldw + r0] : (T)0, y1 = r1 < n ? W[nrp * ldw + r1] : (T)0;
    const T i0 = r0 < n ? (T)1 / Ld[(r0 >> 4) * kDs + (r0 & 15) * 18] : (T)0;
    const T i1 = r1 < n ? (T)1 / Ld[(r1 >> 4) * kDs + (r1 & 15) * 18] : (T)0;
    T x0 = (T)0, x1 = (T)0;
    // rows from the last, a block of 16 at a time (entries L_ir for r < i
    // only, zero otherwise, loaded off the chain); first those of the upper half
#pragma unroll 1
    for (int b = mb - 1; b >= 4; --b) {
      const T* p0 = W + 16 * b * ldw + r0;
      const bool in = r1 >> 4 == b;
      const T* p1 = in ? Ld + b * kDs + (r1 & 15) : W + 16 * b * ldw + min(r1, nrp - 1);
      const int s1 = in ? 17 : ldw;
      T l0[16], l1[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        l0[c] = p0[c * ldw];
        l1[c] = r1 < 16 * b + c ? p1[c * s1] : (T)0;
      }
#pragma unroll
      for (int c = 15; c >= 0; --c) {
        const int i = 16 * b + c;
        if (i >= n) continue;  // uniform
        const T xi = lane_bcast(y1 * i1, i - 64);
        y0 -= l0[c] * xi;
        y1 -= l1[c] * xi;
        x1 = r1 == i ? xi : x1;
      }
    }
#pragma unroll 1
    for (int b = min(mb, 4) - 1; b >= 0; --b) {
      const bool in = r0 >> 4 == b;
      const T* p0 = in ? Ld + b * kDs + (r0 & 15) : W + 16 * b * ldw + min(r0, nrp - 1);
      const int s0 = in ? 17 : ldw;
      T l0[16];
#pragma unroll
      for (int c = 0; c < 16; ++c) l0[c] = r0 < 16 * b + c ? p0[c * s0] : (T)0;
#pragma unroll
      for (int c = 15; c >= 0; --c) {
        const int i = 16 * b + c;
        if (i >= n) continue;  // uniform
        const T xi = lane_bcast(y0 * i0, i);
        y0 -= l0[c] * xi;
        x0 = r0 == i ? xi : x0;
      }
    }
    if (r0 < n) x[r0] = bad ? (T)0 : x0;
    if (r1 < n) x[r1] = bad ? (T)0 : x1;
    if (lane == 0) *bad_out = bad;
  } else {
    if (w == 1) {  // smallest L_jj^2 / S_jj
      unsigned int m = __float_as_uint(3.0e38f);
      for (int j = lane; j < n; j += 64) {
        const T l = Ld[(j >> 4) * kDs + (j & 15) * 18];
        const float ratio = (float)(l * l / dd[j]);
        m = min(m, __float_as_uint(l > (T)0 && ratio == ratio ? fmaxf(ratio, 0.f) : 0.f));
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) m = min(m, (unsigned int)__shfl_xor((int)m, o));
      if (lane == 0) *minr_out = __uint_as_float(m);
    }
    beside();
  }
  __syncthreads();
}

// In-place Cholesky of the packed lower triangle of rows 0..nr-1 of an
// n-column system (nr = n, or n + 1 with the right-hand side appended as row
// n, which then ends as y = L^-1 s; nr <= 256) by at least four wavefronts, in
// panels of 16 columns.  Panel j0: every wavefront that has rows below the 16 x
// 16 diagonal block loads the block (an identity beyond column n) and four
// 16-row blocks, and after a barrier factors and stores its rows (chol16); then
// all update the trailing triangle on the matrix cores, one 16 x 16 tile at a
// time.  Three barriers a panel.  256 systems of up to 234 unknowns, one
// to a CU, on eight wavefronts: 96 us with their solve (one wavefront with
// four rows a lane and entries broadcast through scalar registers, the update
// by dot products in vector registers: 172 us).  invd[j] = 1 / L_jj and piv[j] =
// L_jj^2; a pivot that is not positive or not finite leaves its column
// unscaled (invd 1, piv the pivot) and sets *bad (shared, cleared by the caller).
template <typename T>
__device__ __forceinline__ void packed_panel_factor(T* A, int n_in, int nr_in, T* invd, T* piv, int* bad) {
  const int n = __builtin_amdgcn_readfirstlane(n_in);
  const int nr = __builtin_amdgcn_readfirstlane(nr_in);
  const int tid = threadIdx.x, lane = tid & 63, s = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), nwav = (int)blockDim.x >> 6;
  int badl = 0;
#pragma unroll 1
  for (int j0 = 0; j0 < n; j0 += 16) {
    const int s0 = j0 + 16, below = min(s0, n);  // first row below the panel (row n after a partial one)
    const int i = j0 + s, r = below + 16 * (4 * w + q) + s;
    const bool on = w == 0 || below + 64 * w < nr;
    T ra[16], rb[16];
    if (on) {
      const T* Ai = A + packed_index(min(i, n - 1), j0);
      const T* Ar = A + packed_index(min(r, nr - 1), j0);
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        ra[c] = i < n && c <= s ? Ai[c] : (T)(i >= n && c == s ? 1 : 0);
        rb[c] = r < nr && j0 + c < n ? Ar[c] : (T)0;
      }
    }
    __syncthreads();
    if (on) {
      chol16<T>(ra, rb, badl);
      if (r < nr) {
        T* Ar = A + packed_index(r, j0);
#pragma unroll
        for (int c = 0; c < 16; ++c)
          if (j0 + c < n) Ar[c] = rb[c];
      }
      if (w == 0 && q == 0 && i < n) {
        T* Ai = A + packed_index(i, j0);
#pragma unroll
        for (int c = 0; c < 16; ++c)
          if (c <= s) Ai[c] = ra[c];
      }
    }
    __syncthreads();
    if (s0 < n) {
      // tile (bi, bk), bk <= bi, of the trailing rows s0 .. nr - 1, columns s0 .. n - 1
      const int nbr = (nr - s0 + 15) >> 4, nbc = (n - s0 + 15) >> 4;
      int bi = 0, bk = w;
#pragma unroll 1
      for (;;) {
        while (bi < nbr && bk > min(bi, nbc - 1)) {
          bk -= min(bi, nbc - 1) + 1;
          ++bi;
        }
        if (bi >= nbr) break;
        const T* xr = A + packed_index(min(s0 + 16 * bi + s, nr - 1), j0) + q;
        const T* yr = A + packed_index(min(s0 + 16 * bk + s, n - 1), j0) + q;
        typename Mfma<T>::acc_t acc = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 16; k += 4) acc = Mfma<T>::step(xr[k], yr[k], acc);
        const int k = s0 + 16 * bk + s;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = s0 + 16 * bi + Mfma<T>::row(lane, v);
          if (row < nr && k <= row && k < n) A[packed_index(row, k)] -= acc[v];
        }
        bk += nwav;
      }
    }
    __syncthreads();
  }
  if (badl && lane == 0) *bad = 1;
  for (int j = tid; j < n; j += blockDim.x) {
    const T l = A[packed_index(j, j)];
    const bool ok = l > (T)0 && l < (T)3.0e38;
    invd[j] = ok ? (T)1 / l : (T)1;
    piv[j] = ok ? l * l : l;
  }
  __syncthreads();
}

// Sixteen backward steps i = i_hi, i_hi - 1, ... (i < n) with row i held in
// register set TI: x_i = y_i / L_ii, then y_r -= L_ir x_i on every lane (l:
// L_ir of the lane's four rows, zero unless r < i); x_i is kept by the lane
// of row i.
template <typename T, int TI>
__device__ __forceinline__ void packed_back16(int i_hi, int n, const T (*l)[16], const T* iv, T* y, T* xk,
                                              int lane) {
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const int i = i_hi - c;
    if (i >= n) continue;  // uniform
    const T xi = lane_bcast(y[TI], i & 63) * iv[c];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      y[t] -= l[t][c] * xi;
      xk[t] = lane + 64 * t == i ? xi : xk[t];
    }
  }
}

// L^T x = y on the first wavefront for a packed factor with invd[j] = 1 /
// L_jj (n <= 256; y and x may alias).  Rows r = l + 64 t sit on lane l;
// blocks of 16 rows from the last, whose L entries are loaded before the
// dependent chain.  The other threads return at once (no barrier inside).
template <typename T>
__device__ __forceinline__ void packed_back_solve(const T* A, int n_in, const T* invd, const T* y_in, T* x) {
  if (threadIdx.x >= 64) return;
  const int n = __builtin_amdgcn_readfirstlane(n_in);
  const int lane = threadIdx.x;
  T y[4], xk[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    y[t] = lane + 64 * t < n ? y_in[lane + 64 * t] : (T)0;
    xk[t] = (T)0;
  }
  for (int blk = (n - 1) >> 4; blk >= 0; --blk) {
    T l[4][16], iv[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const int i = 16 * blk + 15 - c, ic = min(i, n - 1);
      iv[c] = invd[ic];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = lane + 64 * t;
        l[t][c] = (r < i && i < n) ? A[packed_index(ic, r)] : (T)0;
      }
    }
    switch (blk >> 2) {  // the set that holds rows 16 blk .. 16 blk + 15
      case 0: packed_back16<T, 0>(16 * blk + 15, n, l, iv, y, xk, lane); break;
      case 1: packed_back16<T, 1>(16 * blk + 15, n, l, iv, y, xk, lane); break;
      case 2: packed_back16<T, 2>(16 * blk + 15, n, l, iv, y, xk, lane); break;
      default: packed_back16<T, 3>(16 * blk + 15, n, l, iv, y, xk, lane); break;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (lane + 64 * t < n) x[lane + 64 * t] = xk[t];
}

// Sixteen forward steps i = i_lo, i_lo + 1, ... (i < n), row i in set TI:
// y_i = b_i / L_ii, then b_r -= L_ri y_i (l: L_ri, zero unless r > i).
template <typename T, int TI>
__device__ __forceinline__ void packed_fwd16(int i_lo, int n, const T (*l)[16], const T* iv, T* b, T* yk,
                                             int lane) {
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const int i = i_lo + c;
    if (i >= n) continue;  // uniform
    const T yi = lane_bcast(b[TI], i & 63) * iv[c];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      b[t] -= l[t][c] * yi;
      yk[t] = lane + 64 * t == i ? yi : yk[t];
    }
  }
}

// L y = b on the first wavefront (the companion of packed_back_solve; b and
// y may alias).
template <typename T>
__device__ __forceinline__ void packed_fwd_solve(const T* A, int n_in, const T* invd, const T* b_in, T* y) {
  if (threadIdx.x >= 64) return;
  const int n = __builtin_amdgcn_readfirstlane(n_in);
  const int lane = threadIdx.x;
  T b[4], yk[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    b[t] = lane + 64 * t < n ? b_in[lane + 64 * t] : (T)0;
    yk[t] = (T)0;
  }
  for (int blk = 0; 16 * blk < n; ++blk) {
    T l[4][16], iv[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const int i = 16 * blk + c, ic = min(i, n - 1);
      iv[c] = invd[ic];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = lane + 64 * t;
        l[t][c] = (r > i && r < n) ? A[packed_index(r, ic)] : (T)0;
      }
    }
    switch (blk >> 2) {
      case 0: packed_fwd16<T, 0>(16 * blk, n, l, iv, b, yk, lane); break;
      case 1: packed_fwd16<T, 1>(16 * blk, n, l, iv, b, yk, lane); break;
      case 2: packed_fwd16<T, 2>(16 * blk, n, l, iv, b, yk, lane); break;
      default: packed_fwd16<T, 3>(16 * blk, n, l, iv, b, yk, lane); break;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (lane + 64 * t < n) y[lane + 64 * t] = yk[t];
}

}  // namespace dpvba
