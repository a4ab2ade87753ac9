// Matrix-core (MFMA) helpers for gfx950.
#pragma once

#include <hip/hip_runtime.h>

namespace dpvba {

typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef double doublex4_t __attribute__((ext_vector_type(4)));

// 16x16x4 matrix-core step D = A B + C: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16]; its v-th accumulator (v = 0..3) holds
// D[row(l, v)][l % 16], with row = 4 (l / 16) + v for float32 and
// row = l / 16 + 4 v for float64 (checked on gfx950).
template <typename T> struct Mfma;
template <> struct Mfma<float> {
  typedef floatx4_t acc_t;
  static __device__ __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};
template <> struct Mfma<double> {
  typedef doublex4_t acc_t;
  static __device__ __forceinline__ acc_t step(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};

// 16 bytes of a row.
template <typename T> struct V16;
template <> struct V16<float> { typedef float type __attribute__((ext_vector_type(4))); };
template <> struct V16<double> { typedef double type __attribute__((ext_vector_type(2))); };

// N entries between registers and a 16-byte aligned row in LDS.
template <typename T, int N>
__device__ __forceinline__ void get_row(const T* row, T* r) {
  constexpr int V = 16 / (int)sizeof(T);
#pragma unroll
  for (int c = 0; c < N; c += V) {
    const typename V16<T>::type v = *reinterpret_cast<const typename V16<T>::type*>(row + c);
#pragma unroll
    for (int u = 0; u < V; ++u) r[c + u] = v[u];
  }
}
template <typename T, int N>
__device__ __forceinline__ void put_row(T* row, const T* r) {
  constexpr int V = 16 / (int)sizeof(T);
#pragma unroll
  for (int c = 0; c < N; c += V) {
    typename V16<T>::type v;
#pragma unroll
    for (int u = 0; u < V; ++u) v[u] = r[c + u];
    *reinterpret_cast<typename V16<T>::type*>(row + c) = v;
  }
}

}  // namespace dpvba
