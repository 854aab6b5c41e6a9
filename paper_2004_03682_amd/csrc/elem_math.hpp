// elem_math.hpp -- the element arithmetic that the reorder and elementwise
// kernels share.  The fused multiply-adds are written out, so that every
// traversal and the fused launches give the same bits (left to the compiler,
// two kernels contract the same expression differently).
#pragma once

#include <hip/hip_runtime.h>

namespace fscc {

__device__ __forceinline__ double2 elem_mul(double2 x, double2 y) {
    return make_double2(__builtin_fma(x.x, y.x, -(x.y * y.y)), __builtin_fma(x.x, y.y, x.y * y.x));
}
__device__ __forceinline__ double elem_mul(double x, double y) { return x * y; }

__device__ __forceinline__ double2 elem_scale(double ar, double ai, double2 s) {
    return make_double2(__builtin_fma(ar, s.x, -(ai * s.y)), __builtin_fma(ar, s.y, ai * s.x));
}
__device__ __forceinline__ double elem_scale(double ar, double, double s) { return ar * s; }

// s + x y
__device__ __forceinline__ double2 elem_add_mul(double2 s, double2 x, double2 y) {
    const double2 z = elem_mul(x, y);
    return make_double2(s.x + z.x, s.y + z.y);
}
__device__ __forceinline__ double elem_add_mul(double s, double x, double y) { return __builtin_fma(x, y, s); }

// a s + o
__device__ __forceinline__ double2 elem_scale_add(double ar, double ai, double2 s, double2 o) {
    const double2 z = elem_scale(ar, ai, s);
    return make_double2(z.x + o.x, z.y + o.y);
}
__device__ __forceinline__ double elem_scale_add(double ar, double, double s, double o) { return __builtin_fma(ar, s, o); }

// o - d x
__device__ __forceinline__ double2 elem_sub(double2 o, double d, double2 x) {
    return make_double2(__builtin_fma(-d, x.x, o.x), __builtin_fma(-d, x.y, o.y));
}
__device__ __forceinline__ double elem_sub(double o, double d, double x) { return __builtin_fma(-d, x, o); }

}  // namespace fscc
