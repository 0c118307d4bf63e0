// Device helpers shared by the kernels that read raw frames: plain or
// non-temporal loads, and the correction of one pixel (Section 6.4).
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace azi {
namespace {

template <bool NT, class T>
__device__ inline T ld(const T* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <class T> struct Pair2;
template <> struct Pair2<double> { using type = double2; };
template <> struct Pair2<float> { using type = float2; };

// (T(raw) - dark) * (1 / norm) from a pair of the storage type, or from a
// 12-byte record (float dark, double 1 / norm) used when every dark value
// is a float: the cast back to double is exact, so both give the same bits.
__device__ inline double corr_apply(double v, const double2& c) { return (v - c.x) * c.y; }
__device__ inline float corr_apply(float v, const float2& c) { return (v - c.x) * c.y; }
__device__ inline double corr_apply(double v, const Corr12& c) {
    const double inv = __hiloint2double((int)c.inv_hi, (int)c.inv_lo);
    return (v - (double)c.dark) * inv;
}
// Dark alone, when the coefficients carry 1 / norm (AZI_STAGE_FOLD): the
// difference of an integer count and a float dark is exact in double.
__device__ inline double corr_apply(double v, float d) { return v - (double)d; }
__device__ inline double corr_apply(double v, double d) { return v - d; }
__device__ inline float corr_apply(float v, float d) { return v - d; }
// An integer dark count of 16 bits: exact in float and double alike.
__device__ inline double corr_apply(double v, uint16_t d) { return v - (double)d; }
__device__ inline float corr_apply(float v, uint16_t d) { return v - (float)d; }
template <class T, class V>
__device__ inline T corr_apply(T v, RunDark<V> d) { return corr_apply(v, d.v); }
template <class C> struct IsRunDark { static constexpr bool value = false; };
template <class V> struct IsRunDark<RunDark<V>> { static constexpr bool value = true; };

}  // namespace
}  // namespace azi
