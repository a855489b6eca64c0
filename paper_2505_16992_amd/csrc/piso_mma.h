// FP32 / FP64 matrix instructions and 16-byte LDS accesses of the fast-diagonalisation kernels.
#pragma once

namespace piso {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

template <typename R>
struct Vec4;
template <>
struct Vec4<float> {
  using T = f32x4;
};
template <>
struct Vec4<double> {
  using T = f64x4;
};

__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Row of the 16-row output tile in which register r of lane group g holds its result, and
// its inverse, the packing order that makes that row 4 g + r in both types: the FP32
// instruction returns row 4 g + r, the FP64 one row 4 r + g.
template <typename R>
constexpr int packed_row(int m) {
  return sizeof(R) == 4 ? m : 4 * (m % 4) + m / 4;
}

template <typename R>
__device__ __forceinline__ typename Vec4<R>::T lds4(const R* p) {
  typename Vec4<R>::T v;
  if constexpr (sizeof(R) == 4) {
    v = *reinterpret_cast<const f32x4*>(p);
  } else {
    const f64x2 a = *reinterpret_cast<const f64x2*>(p), b = *reinterpret_cast<const f64x2*>(p + 2);
    v[0] = a[0];
    v[1] = a[1];
    v[2] = b[0];
    v[3] = b[1];
  }
  return v;
}

template <typename R>
__device__ __forceinline__ void sts4(R* p, typename Vec4<R>::T v) {
  if constexpr (sizeof(R) == 4) {
    *reinterpret_cast<f32x4*>(p) = v;
  } else {
    *reinterpret_cast<f64x2*>(p) = f64x2{v[0], v[1]};
    *reinterpret_cast<f64x2*>(p + 2) = f64x2{v[2], v[3]};
  }
}

}  // namespace piso
