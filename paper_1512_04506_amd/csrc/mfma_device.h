// The 16x16x4 matrix instructions in FP32 and FP64 behind one name, and loads
// of several consecutive entries.  A[i][k] is held by lane i + 16 k, B[k][j]
// by lane j + 16 k; the result's column is lane % 16 in both, its rows differ.
#pragma once
#include "ddamg_internal.h"

namespace ddamg {
namespace dev {

typedef float mm_f4 __attribute__((ext_vector_type(4)));
typedef double mm_d4 __attribute__((ext_vector_type(4)));
template <typename T> struct MmAcc;
template <> struct MmAcc<float> { using type = mm_f4; };
template <> struct MmAcc<double> { using type = mm_d4; };
__device__ inline mm_f4 mm_mfma(float a, float b, mm_f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline mm_d4 mm_mfma(double a, double b, mm_d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// row of the 16x16 result in register v of lane group lg = lane / 16
template <typename T>
__device__ inline int mm_row(int lg, int v) {
  return sizeof(T) == 8 ? lg + 4 * v : 4 * lg + v;
}

// N consecutive entries at the alignment of one (4 or 8 bytes: global loads
// of any width need no more)
template <typename X, int N>
struct __attribute__((packed, aligned(sizeof(X) < 8 ? sizeof(X) : 8))) Run {
  X v[N];
};
template <typename X, int N>
__device__ inline Run<X, N> load_run(const X* p) {
  return *reinterpret_cast<const Run<X, N>*>(p);
}

}  // namespace dev
}  // namespace ddamg
