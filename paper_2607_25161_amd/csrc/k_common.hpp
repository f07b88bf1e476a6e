// Device helpers shared by the mobility and transform kernels.
#pragma once
#include <type_traits>

#include "fsd_impl.hpp"

namespace fsd {

template <typename R>
struct C2;
template <>
struct C2<double> {
  using T = double2;
};
template <>
struct C2<float> {
  using T = float2;
};

template <typename T>
__device__ __forceinline__ T cmul(T a, T b) {
  T r;
  r.x = a.x * b.x - a.y * b.y;
  r.y = a.x * b.y + a.y * b.x;
  return r;
}
template <typename T>
__device__ __forceinline__ T cadd(T a, T b) {
  T r;
  r.x = a.x + b.x;
  r.y = a.y + b.y;
  return r;
}
template <typename T>
__device__ __forceinline__ T csub(T a, T b) {
  T r;
  r.x = a.x - b.x;
  r.y = a.y - b.y;
  return r;
}

// Global-memory accesses through a 32-bit element index i from a base the workgroup shares
// (the caller keeps i sizeof(R) below 2^32), so a load or store takes a 32-bit offset
// instead of a 64-bit address.  stg2 stores the pair p[i], p[i + 1] (i even); ldg4 loads
// p[i .. i + 3] (i a multiple of 4, aligned); ldg2 loads the pair p[i], p[i + 1].
template <typename R>
__device__ __forceinline__ void stg2(R* p, unsigned i, R a, R b) {
  typedef R V2 __attribute__((ext_vector_type(2)));
  const unsigned bytes = i * unsigned(sizeof(R));
  V2 v;
  v.x = a;
  v.y = b;
  *(__attribute__((address_space(1))) V2*)((__attribute__((address_space(1))) char*)p + bytes) = v;
}

template <typename R>
__device__ __forceinline__ R ldg1(const R* p, unsigned i) {
  const unsigned bytes = i * unsigned(sizeof(R));
  return *(__attribute__((address_space(1))) const R*)((__attribute__((address_space(1))) const char*)p + bytes);
}

template <typename R>
__device__ __forceinline__ void ldg4(const R* p, unsigned i, R& a, R& b, R& c, R& d) {
  typedef R V4 __attribute__((ext_vector_type(4)));
  const unsigned bytes = i * unsigned(sizeof(R));
  const V4 v = *(__attribute__((address_space(1))) const V4*)((__attribute__((address_space(1))) const char*)p + bytes);
  a = v.x;
  b = v.y;
  c = v.z;
  d = v.w;
}

template <typename R>
__device__ __forceinline__ void ldg2(const R* p, unsigned i, R& a, R& b) {
  typedef R V2 __attribute__((ext_vector_type(2)));
  const unsigned bytes = i * unsigned(sizeof(R));
  const V2 v = *(__attribute__((address_space(1))) const V2*)((__attribute__((address_space(1))) const char*)p + bytes);
  a = v.x;
  b = v.y;
}

// the FP64 or FP32 pointer of a pair
template <typename R>
__device__ inline const R* pick(const double* a, const float* b);
template <>
__device__ inline const double* pick<double>(const double* a, const float*) {
  return a;
}
template <>
__device__ inline const float* pick<float>(const double*, const float* b) {
  return b;
}

}  // namespace fsd
