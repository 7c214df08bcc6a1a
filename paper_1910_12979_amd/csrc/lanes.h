// What the kernels that march with columns in registers share: moves between
// the lanes of a wavefront, indices and addresses.
#pragma once

#include <hip/hip_runtime.h>

namespace mg {
namespace {

// Index k of a direction of n entries, a few beyond either end: the periodic
// image, or the nearest entry there is (its value is then not used).
__device__ __forceinline__ int fold(int k, int n, int per) {
    if (per) {
        while (k < 0) k += n;
        while (k >= n) k -= n;
        return k;
    }
    return min(max(k, 0), n - 1);
}

// The value of x in the lane below / above (0 at the wavefront's ends): moves
// within the vector registers, no LDS.  Every lane of the wavefront must be
// active.
__device__ __forceinline__ float lane_lo(float x) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_hi(float x) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x130, 0xf, 0xf, true));
}
struct LaneHalves {
    float a, b;
};
__device__ __forceinline__ double lane_lo(double x) {
    const LaneHalves v = __builtin_bit_cast(LaneHalves, x);
    return __builtin_bit_cast(double, LaneHalves{lane_lo(v.a), lane_lo(v.b)});
}
__device__ __forceinline__ double lane_hi(double x) {
    const LaneHalves v = __builtin_bit_cast(LaneHalves, x);
    return __builtin_bit_cast(double, LaneHalves{lane_hi(v.a), lane_hi(v.b)});
}

// Workgroup b of n runs on XCD b mod 8: tile of it such that an XCD's
// workgroups have consecutive tiles, whose windows overlap in its L2.
__device__ __forceinline__ int xcd_order(int b, int n) {
    const int x = b % 8, q = n / 8, r = n % 8;
    return x * q + min(x, r) + b / 8;
}

// Four loaded values, waited for together at this point.
template <typename T>
__device__ __forceinline__ void at_once(T& a, T& b, T& c, T& d) {
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// Element at byte offset o (32 bits: a plane's) of a plane that starts at
// index k * n of a: the plane's address stays in scalar registers.
template <typename T>
__device__ __forceinline__ const T* plane_at(const T* a, int k, size_t n) {
    return a + (size_t)(unsigned)k * n;
}
template <typename T>
__device__ __forceinline__ T at_byte(const T* a, unsigned o) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(a) + o);
}
template <typename T>
__device__ __forceinline__ void put_byte(T* a, unsigned o, T v) {
    *reinterpret_cast<T*>(reinterpret_cast<char*>(a) + o) = v;
}

}  // namespace
}  // namespace mg
