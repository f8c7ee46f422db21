// Matrix-core helpers (gfx950): the 16x16x4 matrix instruction of each element
// type with its operand and result layouts, and tile indices.
#pragma once
#include "rs_device.hpp"

namespace rs {
namespace mf {

__device__ __forceinline__ int wave() { return uni((int)(threadIdx.x >> 6)); }
__device__ __forceinline__ int lane() { return (int)(threadIdx.x & 63); }

// The 16x16x4 matrix instruction of each element type.  Operand layout
// (checked on gfx950 for both): A element (i,k) in lane i + 16k, B element
// (k,j) in lane j + 16k.  Result element (row(r), lane%16) in acc[r] with
// row(r) = lane/16 + 4r for f64 and 4(lane/16) + r for f32.
template <class T>
struct MT;
template <>
struct MT<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mfma(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r) { return (lane() >> 4) + 4 * r; }
};
template <>
struct MT<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mfma(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r) { return 4 * (lane() >> 4) + r; }
};
template <class T>
using v4_t = typename MT<T>::v4;
typedef v4_t<double> d4;

template <class T = double>
__device__ __forceinline__ v4_t<T> zero4() { return v4_t<T>{T(0), T(0), T(0), T(0)}; }

// Row / column of element r of this lane in tile (ti, tj).
template <class T>
__device__ __forceinline__ int trow(int ti, int r) { return 16 * ti + MT<T>::row(r); }
__device__ __forceinline__ int tcol(int tj) { return 16 * tj + (lane() & 15); }

// Lower-triangular tile index t (0 .. T(T+1)/2-1) of a T x T tile grid.
__device__ __forceinline__ void lower_tile(int t, int &ti, int &tj) {
    ti = 0;
    while ((ti + 1) * (ti + 2) / 2 <= t) ++ti;
    tj = t - ti * (ti + 1) / 2;
}

// Orders one wavefront's LDS accesses (no workgroup barrier).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ __forceinline__ double rsq_est(double d) { return __builtin_amdgcn_rsq(d); }
__device__ __forceinline__ float rsq_est(float d) { return __builtin_amdgcn_rsqf(d); }

}  // namespace mf
}  // namespace rs
