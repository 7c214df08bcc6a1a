// Dense coarsest-level inversion shared by the cell-centred and the nodal
// multigrid: the matrix of a level of at most kCoarseMax unknowns, -A plus a
// constant on every entry where the operator is singular, inverted by
// Gauss-Jordan elimination without pivoting (it is symmetric positive
// definite).
//
// Up to kDenseReg unknowns one 256-thread workgroup holds the matrix in
// registers.  Each pivot depends on the one before it, so the time is n times
// the latency of one step (write the pivot row and column to LDS, barrier,
// read them, one reciprocal, update): the step has one barrier and no memory
// access but those two vectors, and four waves (one per SIMD, up to 64
// entries a thread) read them from LDS four times less often than sixteen
// would.  MI355X: 64 unknowns 58 -> 24 us and 80 (nodal) 175 -> 75 us against
// one workgroup on the matrix in LDS or in global memory with two barriers a
// pivot.
// Above it, blocks of kDenseNB pivots: one workgroup inverts the pivot block
// and multiplies its rows by it, then one workgroup per strip of rows updates
// the matrix in place.  420 unknowns: 18.0 -> 0.33 ms, 144 (nodal) 788 -> 115
// us; what is left is two dependent launches a block, 8 and 4 us each.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

#include "devmath.h"
#include "mg_internal.h"

namespace mg {

constexpr int kDenseReg = 128;       // unknowns inverted by one workgroup: 144 take 122 us there (10 x 10 entries a
                                     // thread) against 115 us in blocks, 192 285 against 165 us
constexpr int kDenseNB = 16;         // pivots per block step above that: the block's rows (kDenseNB x n doubles)
                                     // fit the 64 KB partial-sum buffer that every hierarchy has
constexpr int kDenseThreads = 256;
constexpr int kDenseGroup = 64;      // rows assembled at a time

// LDS of one inversion: the S off-diagonal entries of every row (value,
// column), the diagonal, one group of assembled rows, and the pivot row and
// column (two of each).
template <int S>
struct DenseLds {
    double val[S][kDenseReg];
    double diag[kDenseReg];
    double rows[kDenseGroup][kDenseReg + 1];
    __align__(16) double prow[2][kDenseReg];
    __align__(16) double pcol[2][kDenseReg];
    double shift;
    int idx[S][kDenseReg];
};

// Mean of diag[0..n-1] by the first wavefront (fixed order), into *out; the
// caller's barrier follows.
__device__ __forceinline__ void dense_mean(const double* diag, int n, double* out) {
    if (threadIdx.x < 64) {
        double s = 0.0;
        for (int c = threadIdx.x; c < n; c += 64) s += diag[c];
        for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w, 64);
        if (threadIdx.x == 0) *out = s / n;
    }
}

// Pivots q E .. q E + E - 1 for every q: each in code of its own (a compile-
// time index into the registers that hold its row and column).
template <typename F, int... R>
__device__ __forceinline__ void dense_pivots(F&& pivot, int n, int E, std::integer_sequence<int, R...>) {
    for (int q = 0; q * E < n; ++q) (pivot(std::integral_constant<int, R>{}, q), ...);
}

// Build and invert an n x n matrix (n <= 16 E) by 256 threads: thread (ti,
// tj) of 16 x 16 holds the E x E entries from (ti E, tj E).  `row(i, e, &val,
// &col)` gives entry e < S of row i (val 0: none), `diag(i)` its diagonal.
template <int S, int E, typename Row, typename Diag>
__device__ __forceinline__ void dense_invert_reg(int n, int singular, double* __restrict__ M, DenseLds<S>& L, Row row, Diag diag) {
    const int tid = threadIdx.x, i0 = (tid >> 4) * E, j0 = (tid & 15) * E;
    for (int q = 0; q < S; ++q)
        for (int i = tid; i < n; i += kDenseThreads) row(i, q, L.val[q][i], L.idx[q][i]);
    for (int i = tid; i < n; i += kDenseThreads) L.diag[i] = diag(i);
    __syncthreads();
    dense_mean(L.diag, n, &L.shift);
    __syncthreads();
    const double sh = singular ? L.shift : 0.0;
    double a[E][E];
#pragma unroll
    for (int r = 0; r < E; ++r)
#pragma unroll
        for (int c = 0; c < E; ++c) a[r][c] = 0.0;
    for (int g = 0; g < n; g += kDenseGroup) {         // rows g .. assembled in LDS, one thread per row
        const int rows = min(kDenseGroup, n - g);
        for (int e = tid; e < rows * 64; e += kDenseThreads)
            for (int j = e & 63; j < n; j += 64) L.rows[e >> 6][j] = sh;
        __syncthreads();
        if (tid < rows) {
            const int i = g + tid;
            for (int q = 0; q < S; ++q)
                if (L.val[q][i] != 0.0) L.rows[tid][L.idx[q][i]] -= L.val[q][i];
            L.rows[tid][i] += L.diag[i];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const int i = i0 + r - g;
            if (i >= 0 && i < rows) {
#pragma unroll
                for (int c = 0; c < E; ++c)
                    if (j0 + c < n) a[r][c] = L.rows[i][j0 + c];
            }
        }
        __syncthreads();
    }
    // pivot p = q E + R: row p becomes row p / M_pp (1 / M_pp in column p),
    // every other row i subtracts M_ip times it (column p: -M_ip / M_pp)
    int b = 0;
    auto pivot = [&](auto Rc, int q) {
        constexpr int R = decltype(Rc)::value;
        const int p = q * E + R;
        if (p >= n) return;
        const bool pr = i0 == q * E, pc = j0 == q * E;
        if (pr) {
#pragma unroll
            for (int c = 0; c < E; ++c) L.prow[b][j0 + c] = a[R][c];
        }
        if (pc) {
#pragma unroll
            for (int r = 0; r < E; ++r) L.pcol[b][i0 + r] = a[r][R];
        }
        __syncthreads();
        const double inv = qdiv(1.0, L.pcol[b][p]);
        double np[E], f[E];
#pragma unroll
        for (int c = 0; c < E; ++c) np[c] = L.prow[b][j0 + c] * inv;
#pragma unroll
        for (int r = 0; r < E; ++r) f[r] = L.pcol[b][i0 + r];
        if (pc) {
            np[R] = inv;
#pragma unroll
            for (int r = 0; r < E; ++r) a[r][R] = 0.0;
        }
#pragma unroll
        for (int r = 0; r < E; ++r)
#pragma unroll
            for (int c = 0; c < E; ++c) a[r][c] = fma(-f[r], np[c], a[r][c]);
        if (pr) {
#pragma unroll
            for (int c = 0; c < E; ++c) a[R][c] = np[c];
        }
        b ^= 1;
    };
    dense_pivots(pivot, n, E, std::make_integer_sequence<int, E>{});
#pragma unroll
    for (int r = 0; r < E; ++r)
#pragma unroll
        for (int c = 0; c < E; ++c)
            if (i0 + r < n && j0 + c < n) M[(size_t)(i0 + r) * n + j0 + c] = a[r][c];
}

// The same for any n <= kDenseReg (the entries do not depend on E).
template <int S, typename Row, typename Diag>
__device__ __forceinline__ void dense_invert(int n, int singular, double* __restrict__ M, DenseLds<S>& L, Row row, Diag diag) {
    if (n <= 64) dense_invert_reg<S, 4>(n, singular, M, L, row, diag);
    else dense_invert_reg<S, 8>(n, singular, M, L, row, diag);
}

// Row blockIdx.x of the matrix (n > kDenseReg): one 256-thread workgroup per
// row; every workgroup forms the mean diagonal in the same order.
template <int S, typename Row, typename Diag>
__device__ __forceinline__ void dense_build_row(int n, int singular, double* __restrict__ M, Row row, Diag diag) {
    __shared__ double d[kCoarseMax], out[kCoarseMax];
    __shared__ double val[S];
    __shared__ int idx[S];
    __shared__ double shift;
    const int i = blockIdx.x;
    for (int c = threadIdx.x; c < n; c += blockDim.x) d[c] = diag(c);
    for (int q = threadIdx.x; q < S; q += blockDim.x) row(i, q, val[q], idx[q]);
    __syncthreads();
    dense_mean(d, n, &shift);
    __syncthreads();
    for (int c = threadIdx.x; c < n; c += blockDim.x) out[c] = singular ? shift : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 0; q < S; ++q)
            if (val[q] != 0.0) out[idx[q]] -= val[q];
        out[i] += d[i];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < n; c += blockDim.x) M[(size_t)i * n + c] = out[c];
}

// Invert the assembled n x n matrix M (device, n <= kCoarseMax) in place;
// scratch: kDenseNB * n doubles.
hipError_t launch_dense_blocks(double* M, int n, double* scratch, hipStream_t st);

// Coarsest solve by the calling workgroup (NT threads, a multiple of 64):
// rhs[0..n-1] (LDS) in, x[0..n-1] (LDS) = M^-1 (-f') out, f' the input with
// its mean removed and x's mean removed where the operator is singular.  The
// matrix is symmetric: thread lanes take its rows in turn and walk down the
// columns, so every load is of consecutive entries; each row's sum is formed
// in kMatvecParts column ranges, added pairwise, so the value depends on n
// alone.  part: kMatvecParts * n doubles of LDS, mean: one.  Ends with a
// barrier.
constexpr int kMatvecParts = 8;
template <int NT>
__device__ __forceinline__ void dense_solve(int n, int singular, const double* __restrict__ minv, double* rhs,
                                            double* x, double* part, double* mean) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (singular) {
        dense_mean(rhs, n, mean);
        __syncthreads();
        const double m = *mean;
        for (int c = threadIdx.x; c < n; c += NT) rhs[c] = rhs[c] - m;
    }
    __syncthreads();
    const int len = (n + kMatvecParts - 1) / kMatvecParts;
    for (int g = wave; g < kMatvecParts; g += NT / 64) {
        const int c0 = min(g * len, n), c1 = min(c0 + len, n);
        for (int r = lane; r < n; r += 64) {
            double s = 0.0;
            for (int c = c0; c < c1; c += 8) {         // eight loads in flight at a time
                double v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = minv[(size_t)min(c + q, c1 - 1) * n + r];
#pragma unroll
                for (int q = 0; q < 8; ++q) s = fma(-v[q], c + q < c1 ? rhs[c + q] : 0.0, s);
            }
            part[g * n + r] = s;
        }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < n; r += NT)
        x[r] = ((part[r] + part[n + r]) + (part[2 * n + r] + part[3 * n + r])) +
               ((part[4 * n + r] + part[5 * n + r]) + (part[6 * n + r] + part[7 * n + r]));
    __syncthreads();
    if (singular) {
        dense_mean(x, n, mean);
        __syncthreads();
        const double m = *mean;
        for (int c = threadIdx.x; c < n; c += NT) x[c] = x[c] - m;
        __syncthreads();
    }
}

}  // namespace mg
