// Device helpers of the z-marching kernels: access to a tile's rows in one
// plane of a field, and arithmetic without the compiler's extra steps.
#pragma once

#include <hip/hip_runtime.h>

namespace ptk {
namespace {

template <typename T>
__device__ __forceinline__ T nanmax(T m, T v) {
    // maximum that lets a NaN through (divergence must not be hidden)
    return (v > m || v != v) ? v : m;
}

// Larger of two values as one instruction (fmax would first quiet both
// operands, one more instruction each, since it cannot see where they come
// from; the results are the same).
__device__ __forceinline__ double max1(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float max1(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ double min1(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float min1(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// 1 / b for quot: the instruction's estimate y (relative error e below 2^-23)
// by one iteration of third order, y (1 + e + e^2), which leaves 2^-69.
__device__ __forceinline__ double inverse(double b) {
    const double y = __builtin_amdgcn_rcp(b);
    const double e = __builtin_fma(-b, y, 1.0);
    return __builtin_fma(__builtin_fma(e, e, e), y, y);
}

// a / b by an iteration on the reciprocal and a corrected quotient, without
// the rescaling of the operands that the division has.  Within one unit in
// the last place of the division (two where the dividend is so small that its
// residual is subnormal) for divisors from 2^-1022 to 2^1022, in FP32 from
// 2^-126 to 2^126; infinities, zeros and NaN come out as from the division.
// Outside, the reciprocal leaves the exponent range and the result is wrong.
// In FP64 no quantity of a run comes near the ends; in FP32 a field's value
// can (a permeability goes with the cube of a porosity): see quot_field.
__device__ __forceinline__ double quot(double a, double b) {
    const double y = inverse(b);
    const double q = a * y;
    return __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-b, q, a), y, q), b, a);
}
// Two quotients by the same divisor.
__device__ __forceinline__ void quot2(double a, double b, double d, double& qa, double& qb) {
    const double y = inverse(d);
    const double p = a * y, q = b * y;
    qa = __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-d, p, a), y, p), d, a);
    qb = __builtin_amdgcn_div_fixup(__builtin_fma(__builtin_fma(-d, q, b), y, q), d, b);
}
__device__ __forceinline__ float quot(float a, float b) {
    float y = __builtin_amdgcn_rcpf(b);
    y = __builtin_fmaf(__builtin_fmaf(-b, y, 1.0f), y, y);
    const float q = a * y;
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-b, q, a), y, q), b, a);
}

// A quotient by a value of a field: in FP32 the division (0.5 % of a mixed
// solve at 95^3).
__device__ __forceinline__ double quot_field(double a, double b) { return quot(a, b); }
__device__ __forceinline__ float quot_field(float a, float b) { return a / b; }

// A copy in a register of its own: the queue moves out of the registers a
// plane was loaded into, which then take the loads after next.  (Left to
// itself the compiler loads into other registers and copies at the end of a
// round, which waits for loads just issued.)
__device__ __forceinline__ double fresh(double v) {
    double r;
    asm("v_mov_b64 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ float fresh(float v) {
    float r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// Buffer access to a tile's rows in one plane of a field: their address and
// size are wave-uniform (scalar registers), a lane brings its byte offset in
// them.  A lane with offset OFF_NONE, or any lane where the size is
// given as 0, loads 0 and stores nothing, so that neither the rim of a field
// needs a branch or a select: every step of a wave issues the same number of
// loads and stores, and the wait for a plane's loads need not cover the
// stores and loads issued after them.
using u32 = unsigned int;
constexpr u32 OFF_NONE = 0x80000000u;   // beyond any tile (the rows of a tile hold less than 2 GiB)
constexpr int RSRC_FLAGS = 0x00020000;  // raw 32-bit data
constexpr int NONTEMPORAL = 2;

template <int AUX = 0, typename T>
__device__ __forceinline__ T ldp(const T* rows, u32 bytes, u32 off) {
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(rows), 0, (int)bytes, RSRC_FLAGS);
    if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, AUX));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, AUX));
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <int AUX = 0, typename T>
__device__ __forceinline__ void stp(T* rows, u32 bytes, u32 off, T v) {
    const auto r = __builtin_amdgcn_make_buffer_rsrc(rows, 0, (int)bytes, RSRC_FLAGS);
    if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off, 0, AUX);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(u32, v), r, (int)off, 0, AUX);
}

}  // namespace
}  // namespace ptk
