// Device arithmetic shared by every kernel that forms face coefficients or
// Gauss-Seidel updates, so that a quantity computed by different kernels
// (stored coefficient arrays, coefficients recomputed inside a sweep, single
// or batched launches) is always the same bit pattern.
#pragma once

#include <hip/hip_runtime.h>

namespace mg {

// x / y for y > 0 finite: hardware reciprocal, one Newton step, one residual
// correction (Markstein's form).  Within one ulp of the IEEE quotient and far
// cheaper than the correctly rounded division sequence, which dominated the
// FP64 sweeps.
__device__ __forceinline__ double qdiv(double x, double y) {
    double r = __builtin_amdgcn_rcp(y);
    const double e = fma(-y, r, 1.0);
    r = fma(r, e, r);
    const double q = x * r;
    const double rem = fma(-y, q, x);
    return fma(r, rem, q);
}

// FP32 (the inner cycle of the mixed-precision solve, whose error the FP64
// refinement removes): hardware reciprocal with one Newton step, then one
// multiply; a few ulp at most instead of the correctly rounded sequence.
__device__ __forceinline__ float qdiv(float x, float y) {
    float r = __builtin_amdgcn_rcpf(y);
    const float e = __builtin_fmaf(-y, r, 1.0f);
    r = __builtin_fmaf(r, e, r);
    return x * r;
}

// qdiv with its reciprocal apart, for a divisor that is used several times:
// qdiv(x, y) == qdiv_by(x, y, qrecip(y)) bit for bit.
__device__ __forceinline__ double qrecip(double y) {
    const double r = __builtin_amdgcn_rcp(y);
    const double e = fma(-y, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ double qdiv_by(double x, double y, double r) {
    const double q = x * r;
    const double rem = fma(-y, q, x);
    return fma(r, rem, q);
}
__device__ __forceinline__ float qrecip(float y) {
    const float r = __builtin_amdgcn_rcpf(y);
    const float e = __builtin_fmaf(-y, r, 1.0f);
    return __builtin_fmaf(r, e, r);
}
__device__ __forceinline__ float qdiv_by(float x, float, float r) { return x * r; }

// A row of 4 values of 256 threads (1-D, or 64 x 4) reduced to out[0..3]: [0],
// [1], [3] summed, [2] the maximum, by the binary tree whose first step adds
// thread t + 128 to thread t.  The first two steps read LDS after one barrier
// and the rest stay in the first wavefront: what bounds the reductions, each a
// launch of one workgroup in the chain of a cycle, is that chain (with a
// barrier a step a reduction of 64 rows took 3.4 us, now 2.6).
__device__ __forceinline__ double tree64(double v, bool maximum) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const double o = __shfl_down(v, s);
        v = maximum ? fmax(v, o) : v + o;
    }
    return v;
}
__device__ inline void reduce_row256(double v0, double v1, double v2, double v3, double* out) {
    __shared__ double sh[4][256];
    const int t = threadIdx.y * blockDim.x + threadIdx.x;
    sh[0][t] = v0;
    sh[1][t] = v1;
    sh[2][t] = v2;
    sh[3][t] = v3;
    __syncthreads();
    if (t >= 64) return;
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double a = sh[q][t], b = sh[q][t + 128], c = sh[q][t + 64], d = sh[q][t + 192];
        v[q] = tree64(q == 2 ? fmax(fmax(a, b), fmax(c, d)) : (a + b) + (c + d), q == 2);
    }
    if (t == 0) {
        out[0] = v[0];
        out[1] = v[1];
        out[2] = v[2];
        out[3] = v[3];
    }
}

// Divisions of the fused sweep: qdiv in FP64; in FP32 (the sweeps of the
// inner cycle of a mixed-precision solve, a preconditioner whose error the
// FP64 refinement removes) the hardware reciprocal times x, within 2 ulp,
// two instructions fewer per division in a kernel bound by instruction issue.
__device__ __forceinline__ double pdiv(double x, double y) { return qdiv(x, y); }
__device__ __forceinline__ float pdiv(float x, float y) { return x * __builtin_amdgcn_rcpf(y); }
// pdiv(x, y) == qdiv_by(x, y, precip(y))
__device__ __forceinline__ double precip(double y) { return qrecip(y); }
__device__ __forceinline__ float precip(float y) { return __builtin_amdgcn_rcpf(y); }

}  // namespace mg
