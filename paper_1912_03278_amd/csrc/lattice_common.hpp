// Per-site building blocks shared by the tiled and the LDS-resident lattice
// kernels: vector accesses of the state arrays and the FP64 action terms.
#pragma once

#include "device_common.hpp"

namespace ihmc {

template <typename T>
__device__ __forceinline__ T neg_if(T v, int sign) {
  return sign < 0 ? -v : v;
}

// Four consecutive state values (16 bytes for FP32, 32 bytes for FP64).
template <typename T>
__device__ __forceinline__ void ld4(const T* __restrict__ p, T (&v)[4]);
template <>
__device__ __forceinline__ void ld4<float>(const float* __restrict__ p, float (&v)[4]) {
  const float4 q = *reinterpret_cast<const float4*>(p);
  v[0] = q.x;
  v[1] = q.y;
  v[2] = q.z;
  v[3] = q.w;
}
template <>
__device__ __forceinline__ void ld4<double>(const double* __restrict__ p, double (&v)[4]) {
  const double2 a = reinterpret_cast<const double2*>(p)[0];
  const double2 b = reinterpret_cast<const double2*>(p)[1];
  v[0] = a.x;
  v[1] = a.y;
  v[2] = b.x;
  v[3] = b.y;
}
// The state arrays that the chain table points to live in global memory.
// Accessing them through pointers of the global address space lets the
// compiler use global rather than flat memory instructions: a flat access
// counts as an LDS access too, so every wait for LDS data would also wait for
// the global loads still in flight.
template <class T>
using gmem = __attribute__((address_space(1))) T;
typedef float vf4 __attribute__((ext_vector_type(4)));
typedef double vd2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ void ld4g(const gmem<T>* p, T (&v)[4]);
template <>
__device__ __forceinline__ void ld4g<float>(const gmem<float>* p, float (&v)[4]) {
  const vf4 q = *(const gmem<vf4>*)p;
  v[0] = q.x;
  v[1] = q.y;
  v[2] = q.z;
  v[3] = q.w;
}
template <>
__device__ __forceinline__ void ld4g<double>(const gmem<double>* p, double (&v)[4]) {
  const vd2 a = ((const gmem<vd2>*)p)[0];
  const vd2 b = ((const gmem<vd2>*)p)[1];
  v[0] = a.x;
  v[1] = a.y;
  v[2] = b.x;
  v[3] = b.y;
}
template <typename T>
__device__ __forceinline__ void st4g(gmem<T>* p, const T (&v)[4]);
template <>
__device__ __forceinline__ void st4g<float>(gmem<float>* p, const float (&v)[4]) {
  *(gmem<vf4>*)p = vf4{v[0], v[1], v[2], v[3]};
}
template <>
__device__ __forceinline__ void st4g<double>(gmem<double>* p, const double (&v)[4]) {
  ((gmem<vd2>*)p)[0] = vd2{v[0], v[1]};
  ((gmem<vd2>*)p)[1] = vd2{v[2], v[3]};
}

template <typename T>
__device__ __forceinline__ void st4(T* __restrict__ p, const T (&v)[4]);
template <>
__device__ __forceinline__ void st4<float>(float* __restrict__ p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
template <>
__device__ __forceinline__ void st4<double>(double* __restrict__ p, const double (&v)[4]) {
  reinterpret_cast<double2*>(p)[0] = make_double2(v[0], v[1]);
  reinterpret_cast<double2*>(p)[1] = make_double2(v[2], v[3]);
}

// FP64 action and estimator terms of one site of the stored field: the integer
// stencil weights are exact, C and sqrt(J') are the true FP64 constants.  With u =
// Kt psi (nb: the neighbours' part) and y = sqrt(J') u + hw,
//   s     S-density   1/2 psi u - psi h'/sqrt(J') - log cosh(y),   ut   u tanh(y)
// or, in the shifted form (b0 = 0, hw = h'),
//   s     1/2 psi u - log cosh(y),                                 ut   y tanh(y).
// A quad may reach into the row padding, a column into the plane padding: such
// sites take no_site().
//
// These terms and their sums bound the last pass on large lattices by VALU issue
// (914 instructions a wave of 256 sites, 91 % of the cycles on 8192^2 FP32, h = 0; an FP64
// operation holds a SIMD for five cycles, a move or select for three to five).  So
// no division is scaled, a term that is zero for the chain is left out, a site's
// terms are added up before the next one starts (65 registers instead of 84: seven
// waves a SIMD instead of five) and the tiled passes hold the coefficients in
// scalar registers.  Last pass: 4096^2 FP32 121.7 -> 111.0 us, 1024^2 18.8 -> 18.0,
// 128^3 26.8 -> 24.9, 64^3 15.3 -> 14.7; a trajectory of 8^2 FP64 (resident) 9.45 ->
// 9.08.  The values are the same to the bit.
struct SiteAction {
  double s, psi, ut, psih;
};

template <bool SGPR>
__device__ __forceinline__ SiteAction site_action(const ChainDev& cd, double v, double nb, int64_t idx) {
  const double u = cd.C * v + nb;
  const double y = __builtin_fma(cd.sqJ, u, cd.hw);
  double lc, th;
  logcosh_tanh<SGPR>(y, lc, th);
  double hpx = cd.hp0, bx = cd.b0;
  if (cd.h_kind == 2) {
    hpx = cd.hp[idx];
    bx = hpx / cd.sqJ;
  }
  return SiteAction{0.5 * v * u - v * bx - lc, v, (cd.form == FORM_SHIFTED ? y : u) * th, v * hpx};
}

__device__ __forceinline__ SiteAction no_site() { return SiteAction{0.0, 0.0, 0.0, 0.0}; }

}  // namespace ihmc
