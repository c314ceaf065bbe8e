// Device views of the particle state and of its adjoint (structure of arrays,
// rows x[D], v[D], C[D*D], G[D*D] of stride ntot), shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ddm_kernels.hpp"

namespace ddm {

// Position storage: 32-bit fixed point in FP32 (resolution 2^-32 of the unit
// domain, 60x finer than float near x = 0.5, and cell indices come out of
// integer arithmetic), plain double in FP64.
template <typename T> struct Pos;
template <> struct Pos<float> {
  using X = uint32_t;
  // x n - 1/2 in units of 2^-32, in 32-bit halves: x n has the integer part hi
  // and the fraction lo, so its cell is hi - 1 below the half and hi above it
  // (-1, that is 2^32 - 1 unsigned, left of the grid).
  static __device__ __forceinline__ bool cell(X xr, const KCfg& c, int& base, float& f) {
    const uint32_t hi = xr >> (32 - c.nlog2), lo = xr << c.nlog2;
    const uint32_t b = hi - 1u + (lo >> 31);
    if (b > (uint32_t)(c.n - 3)) return false;
    base = (int)b;
    f = 0.5f + (float)(lo ^ 0x80000000u) * 2.3283064365386963e-10f;
    return true;
  }
  static __device__ __forceinline__ double real(X xr) { return (double)xr * 2.3283064365386963e-10; }
  static __device__ __forceinline__ X advance(X xr, float d, bool& ok) {
    const float q = rintf(d * 4294967296.0f);
    ok = fabsf(q) < 1073741824.0f;
    return ok ? xr + (uint32_t)(int32_t)q : xr;
  }
  static __device__ __forceinline__ X from_real(double x) {
    const double q = rint(x * 4294967296.0);
    return q <= 0.0 ? 0u : (q >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)q);
  }
  static __device__ __forceinline__ unsigned long long key(X xr) { return (unsigned long long)xr; }
  static __device__ __forceinline__ double unkey(unsigned long long k) { return (double)k * 2.3283064365386963e-10; }
  // the stored position in a place for a T, and back
  static __device__ __forceinline__ float hold(X xr) { return __uint_as_float(xr); }
  static __device__ __forceinline__ X held(float h) { return __float_as_uint(h); }
};
template <> struct Pos<double> {
  using X = double;
  static __device__ __forceinline__ bool cell(X xr, const KCfg& c, int& base, double& f) {
    const double xs = xr * c.inv_dx;
    const double bf = floor(xs - 0.5);
    if (!(bf >= 0.0 && bf <= (double)(c.n - 3))) return false;
    base = (int)bf;
    f = xs - bf;
    return true;
  }
  static __device__ __forceinline__ double real(X xr) { return xr; }
  static __device__ __forceinline__ X advance(X xr, double d, bool& ok) { ok = true; return xr + d; }
  static __device__ __forceinline__ X from_real(double x) { return x; }
  static __device__ __forceinline__ unsigned long long key(X xr) { return (unsigned long long)__double_as_longlong(xr); }
  static __device__ __forceinline__ double unkey(unsigned long long k) { return __longlong_as_double((long long)k); }
  static __device__ __forceinline__ double hold(X xr) { return xr; }
  static __device__ __forceinline__ X held(double h) { return h; }
};

// A pointer that is the same for the whole wave, held in scalar registers: the
// empty asm hides how it was formed, so that the compiler does not add its
// parts to the lane's offset first (64-bit vector arithmetic for every access)
// but indexes it with one 32-bit lane offset.
template <typename T> using Global = __attribute__((address_space(1))) T;
template <typename T> __device__ __forceinline__ Global<T>* scalar_base(T* p) {
  Global<T>* q = (Global<T>*)p;
#ifdef __HIP_DEVICE_COMPILE__
  asm("" : "+s"(q));     // (the host pass knows no scalar registers)
#endif
  return q;
}

// With a view shifted to the first slot of a workgroup (at()) and the thread
// as the index, all rows share one lane offset.
template <typename T, int D> struct P {
  T* s;
  int64_t ntot;
  using X = typename Pos<T>::X;
  __device__ __forceinline__ P at(int64_t p0) const { return P{s + p0, ntot}; }
  __device__ __forceinline__ Global<X>& xr(int a, int64_t p) const { return scalar_base(reinterpret_cast<X*>(s) + (int64_t)a * ntot)[p]; }
  __device__ __forceinline__ Global<T>& v(int a, int64_t p) const { return scalar_base(s + (int64_t)(D + a) * ntot)[p]; }
  __device__ __forceinline__ Global<T>& C(int a, int b, int64_t p) const { return scalar_base(s + (int64_t)(2 * D + a * D + b) * ntot)[p]; }
  __device__ __forceinline__ Global<T>& G(int a, int b, int64_t p) const {
    return scalar_base(s + (int64_t)(2 * D + D * D + a * D + b) * ntot)[p];
  }
};
// Adjoint states hold plain T in every row.
template <typename T, int D> struct Adj {
  T* s;
  int64_t ntot;
  __device__ __forceinline__ Adj at(int64_t p0) const { return Adj{s + p0, ntot}; }
  __device__ __forceinline__ Global<T>& x(int a, int64_t p) const { return scalar_base(s + (int64_t)a * ntot)[p]; }
  __device__ __forceinline__ Global<T>& v(int a, int64_t p) const { return scalar_base(s + (int64_t)(D + a) * ntot)[p]; }
  __device__ __forceinline__ Global<T>& C(int a, int b, int64_t p) const { return scalar_base(s + (int64_t)(2 * D + a * D + b) * ntot)[p]; }
  __device__ __forceinline__ Global<T>& G(int a, int b, int64_t p) const {
    return scalar_base(s + (int64_t)(2 * D + D * D + a * D + b) * ntot)[p];
  }
};

template <typename T, int D>
__device__ __forceinline__ P<T, D> pv(const void* s, int64_t ntot) {
  return P<T, D>{const_cast<T*>(static_cast<const T*>(s)), ntot};
}
template <typename T, int D>
__device__ __forceinline__ Adj<T, D> av(const void* s, int64_t ntot) {
  return Adj<T, D>{const_cast<T*>(static_cast<const T*>(s)), ntot};
}

}  // namespace ddm
