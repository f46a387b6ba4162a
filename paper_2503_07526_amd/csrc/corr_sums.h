// corr_sums.h -- sample arithmetic and sums of every (sample, accumulator) kind,
// shared by the per-step push kernels and the multi-step push.
#ifndef CORR_SUMS_H
#define CORR_SUMS_H

#include <hip/hip_runtime.h>

#include "corr_internal.h"

namespace corr {

template <int K> struct KT;
template <> struct KT<K_F32_F64>    { using S = float;   using A = double;  static constexpr int NP = 1; };
template <> struct KT<K_F32_KAHAN>  { using S = float;   using A = float;   static constexpr int NP = 2; };
template <> struct KT<K_F32_F32>    { using S = float;   using A = float;   static constexpr int NP = 1; };
template <> struct KT<K_F64_F64>    { using S = double;  using A = double;  static constexpr int NP = 1; };
template <> struct KT<K_CF32_F64>   { using S = float2;  using A = double2; static constexpr int NP = 1; };
template <> struct KT<K_CF32_KAHAN> { using S = float2;  using A = float2;  static constexpr int NP = 2; };
template <> struct KT<K_CF32_F32>   { using S = float2;  using A = float2;  static constexpr int NP = 1; };
template <> struct KT<K_CF64_F64>   { using S = double2; using A = double2; static constexpr int NP = 1; };

// Sample arithmetic used by the block average (sum in push order, then / m).
__device__ __forceinline__ float sadd(float a, float b) { return a + b; }
__device__ __forceinline__ double sadd(double a, double b) { return a + b; }
__device__ __forceinline__ float2 sadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 sadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float sdiv(float a, int m) { return a / (float)m; }
__device__ __forceinline__ double sdiv(double a, int m) { return a / (double)m; }
__device__ __forceinline__ float2 sdiv(float2 a, int m) { return make_float2(a.x / (float)m, a.y / (float)m); }
__device__ __forceinline__ double2 sdiv(double2 a, int m) { return make_double2(a.x / (double)m, a.y / (double)m); }
template <typename S> __device__ __forceinline__ S szero();
template <> __device__ __forceinline__ float szero<float>() { return 0.0f; }
template <> __device__ __forceinline__ double szero<double>() { return 0.0; }
template <> __device__ __forceinline__ float2 szero<float2>() { return make_float2(0.0f, 0.0f); }
template <> __device__ __forceinline__ double2 szero<double2>() { return make_double2(0.0, 0.0); }

// sum += x * conj(r) in the accumulator precision of kind K.  The compensated
// form is Kahan summation with the product folded into the first step:
// y = x*r - c (one rounding), t = h + y, c = (t - h) - y, h = t; the true sum is
// h - c.
template <int K> struct Acc;
template <> struct Acc<K_F32_F64> {
    static __device__ __forceinline__ void add(double &h, double &, float x, float r)
    { h = __builtin_fma((double)x, (double)r, h); }
};
template <> struct Acc<K_F32_KAHAN> {
    static __device__ __forceinline__ void add(float &h, float &c, float x, float r)
    {
        float y = __builtin_fmaf(x, r, -c);
        float t = h + y;
        c = (t - h) - y;
        h = t;
    }
};
template <> struct Acc<K_F32_F32> {
    static __device__ __forceinline__ void add(float &h, float &, float x, float r)
    { h = __builtin_fmaf(x, r, h); }
};
template <> struct Acc<K_F64_F64> {
    static __device__ __forceinline__ void add(double &h, double &, double x, double r)
    { h = __builtin_fma(x, r, h); }
};
template <> struct Acc<K_CF32_F64> {
    static __device__ __forceinline__ void add(double2 &h, double2 &, float2 x, float2 r)
    {
        const double xr = x.x, xi = x.y, rr = r.x, ri = r.y;
        h.x = __builtin_fma(xr, rr, __builtin_fma(xi, ri, h.x));
        h.y = __builtin_fma(xi, rr, __builtin_fma(-xr, ri, h.y));
    }
};
template <> struct Acc<K_CF32_KAHAN> {
    static __device__ __forceinline__ void add(float2 &h, float2 &c, float2 x, float2 r)
    {
        float yr = __builtin_fmaf(x.x, r.x, __builtin_fmaf(x.y, r.y, -c.x));
        float yi = __builtin_fmaf(x.y, r.x, __builtin_fmaf(-x.x, r.y, -c.y));
        float tr = h.x + yr;
        float ti = h.y + yi;
        c.x = (tr - h.x) - yr;
        c.y = (ti - h.y) - yi;
        h.x = tr;
        h.y = ti;
    }
};
template <> struct Acc<K_CF32_F32> {
    static __device__ __forceinline__ void add(float2 &h, float2 &, float2 x, float2 r)
    {
        h.x = __builtin_fmaf(x.x, r.x, __builtin_fmaf(x.y, r.y, h.x));
        h.y = __builtin_fmaf(x.y, r.x, __builtin_fmaf(-x.x, r.y, h.y));
    }
};
template <> struct Acc<K_CF64_F64> {
    static __device__ __forceinline__ void add(double2 &h, double2 &, double2 x, double2 r)
    {
        h.x = __builtin_fma(x.x, r.x, __builtin_fma(x.y, r.y, h.x));
        h.y = __builtin_fma(x.y, r.x, __builtin_fma(-x.x, r.y, h.y));
    }
};

} // namespace corr

#endif
