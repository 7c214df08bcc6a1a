// Bottom of the V-cycle in one workgroup (gfx950).
//
// A coarse level has at most a few thousand cells and the per-colour kernels,
// residual+restriction, coarsest solve and prolongation would each be a
// launch of a few microseconds that keeps a handful of CUs busy.  Here one
// workgroup runs the whole V-cycle from such a level down to the coarsest and
// back, with a barrier between dependent steps.
//
// Per cell the arithmetic is exactly that of the per-level kernels (same
// expressions, same face order, same summation order in the restriction and
// the coarsest solve), so a bottom launch gives the same bits as the
// launches it replaces.  The batched form runs one workgroup per problem.
//
// Every thread owns the same cells throughout and holds their six face
// coefficients, diagonal, its reciprocal, right-hand side and neighbour
// offsets in registers, loaded once; only phi is in LDS, one array per colour
// so that the reads of a wavefront are consecutive (a colour's cells alone
// are every other word, which halves the LDS rate).  A colour phase is then
// bound by its barrier and the latency of one update, not by 12 loads and 50
// index instructions a cell.  512 threads: two waves per SIMD leave each 256
// registers, which eight cells in FP64 take.  From 16^3 down, MI355X: 33 -> 21
// us in FP64 and 36 -> 18 us in FP32, in the 256^3 solve (caches cold) 39 ->
// 25 us, against 1024 threads with everything in LDS or global memory.
#include <hip/hip_runtime.h>

#include "dense.h"
#include "devmath.h"
#include "mg_internal.h"

namespace mg {
namespace {

// Coarsest level (dense_solve): F in, P out, n values each.
template <typename T, int NT>
__device__ void b_coarse(int n, int singular, const double* __restrict__ minv, const T* F, T* P, double* rhs,
                         double* x, double* part, double* mean) {
    for (int c = threadIdx.x; c < n; c += NT) rhs[c] = (double)F[c];
    __syncthreads();
    dense_solve<NT>(n, singular, minv, rhs, x, part, mean);
    for (int c = threadIdx.x; c < n; c += NT) P[c] = (T)x[c];
    __syncthreads();
}

constexpr int kBottomThreads = 512;

// A colour's cells of a level (every smoothed level has even sides) are
// numbered ((k ny + j) nx/2 + ih), i = 2 ih + ((j + k + colour) & 1); phi of
// colour c is at P + c * half.  The neighbours of a cell are all of the other
// colour: in y and z at the same ih, in x at ih and at ih - 1 or ih + 1.
struct CellAt {
    int i, j, k, row;          // row = k ny + j
    unsigned nb[3];            // neighbour numbers in the other colour, low and high in 16 bits each
    int gx, gy, gz;            // natural indices of the cells whose low faces are this cell's high faces
};

template <typename T>
__device__ __forceinline__ CellAt cell_at(const BottomLevel<T>& lv, int c, int e) {
    const int nx = lv.nx, ny = lv.ny, nz = lv.nz, hx = nx >> 1;
    CellAt q;
    int ih;
    small_divmod(e, hx, q.row, ih);
    small_divmod(q.row, ny, q.k, q.j);
    const int j = q.j, k = q.k, s = (j + k + c) & 1;
    q.i = 2 * ih + s;
    const int im = ih > 0 ? ih - 1 : hx - 1, ip = ih < hx - 1 ? ih + 1 : 0;
    const int jm = j > 0 ? j - 1 : ny - 1, jp = j < ny - 1 ? j + 1 : 0;
    const int km = k > 0 ? k - 1 : nz - 1, kp = k < nz - 1 ? k + 1 : 0;
    q.nb[0] = (unsigned)(q.row * hx + (s ? ih : im)) | (unsigned)(q.row * hx + (s ? ip : ih)) << 16;
    q.nb[1] = (unsigned)((k * ny + jm) * hx + ih) | (unsigned)((k * ny + jp) * hx + ih) << 16;
    q.nb[2] = (unsigned)((km * ny + j) * hx + ih) | (unsigned)((kp * ny + j) * hx + ih) << 16;
    q.gx = q.row * nx + (s ? 2 * ip : q.i + 1);
    q.gy = (k * ny + jp) * nx + q.i;
    q.gz = (kp * ny + j) * nx + q.i;
    return q;
}

template <typename T>
__device__ __forceinline__ void cell_coeffs(const BottomLevel<T>& lv, const CellAt& q, T (&b)[6]) {
    const int g = q.row * lv.nx + q.i;
    b[0] = lv.bx[g];
    b[1] = lv.bx[q.gx];
    b[2] = lv.by[g];
    b[3] = lv.by[q.gy];
    b[4] = lv.bz[g];
    b[5] = lv.bz[q.gz];
}

template <typename T>
__device__ __forceinline__ T face_sum(const T (&b)[6]) {
    T d = b[0] + b[1];
    d = d + b[2];
    d = d + b[3];
    d = d + b[4];
    return d + b[5];
}

// The update of one cell from its neighbours O (the other colour's phi).
template <typename T>
__device__ __forceinline__ T cell_update(const T (&b)[6], const unsigned (&n)[3], const T* O, T h2, T f, T den, T rec) {
    T num = b[0] * O[n[0] & 0xffff];
    num = num + b[1] * O[n[0] >> 16];
    num = num + b[2] * O[n[1] & 0xffff];
    num = num + b[3] * O[n[1] >> 16];
    num = num + b[4] * O[n[2] & 0xffff];
    num = num + b[5] * O[n[2] >> 16];
    return qdiv_by(num - h2 * f, den, rec);
}

// f - L phi of one cell; dg: its boundary diagonal (kBnd).
template <bool kBnd, typename T>
__device__ __forceinline__ T cell_residual(const T (&b)[6], const unsigned (&n)[3], const T* O, T pc, T f, T dg, T ih2) {
    T s = b[0] * (O[n[0] & 0xffff] - pc);
    s = s + b[1] * (O[n[0] >> 16] - pc);
    s = s + b[2] * (O[n[1] & 0xffff] - pc);
    s = s + b[3] * (O[n[1] >> 16] - pc);
    s = s + b[4] * (O[n[2] & 0xffff] - pc);
    s = s + b[5] * (O[n[2] >> 16] - pc);
    if (kBnd) s = s - dg * pc;
    return f - s * ih2;
}

// threadIdx.x as a value of its own: the cells' coordinates decoded from it
// late are decoded again instead of being held since the start.
__device__ __forceinline__ int own_thread() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The first level's cells of a thread: e = threadIdx.x + m * kBottomThreads
// of each colour, m < K.  In LDS: phi (P), the residual (R) and, with outflow
// sides (kBnd), the boundary diagonal (G), each by colour.
template <typename T, int K, bool kBnd>
struct Owned {
    // eight cells in FP64 have no registers left for the reciprocals of their diagonals
    static constexpr bool kRec = sizeof(T) == 4 || K < 4;
    T b[2][K][6];              // x low, x high, y low, ...
    T rec[2][kRec ? K : 1];    // reciprocal of the diagonal
    T f[2][K];                 // right-hand side
    unsigned nb[2][K][3];
    int half;

    __device__ __forceinline__ void load(const BottomLevel<T>& lv, const T* __restrict__ F, T* P, T* G) {
        half = (lv.nx >> 1) * lv.ny * lv.nz;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int m = 0; m < K; ++m) {
                const int e = threadIdx.x + m * kBottomThreads;
                const CellAt q = cell_at(lv, c, min(e, half - 1));
                cell_coeffs(lv, q, b[c][m]);
                f[c][m] = F[q.row * lv.nx + q.i];
                for (int d = 0; d < 3; ++d) nb[c][m][d] = q.nb[d];
                if (kBnd && e < half) G[c * half + e] = bnd_diag(lv.bnd, q.i, q.j, q.k, lv.nx, lv.ny, lv.nz);
                if (e < half) P[c * half + e] = T(0);
            }
        if constexpr (kRec) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int m = 0; m < K; ++m) {
                    const T d = diagonal(c, m, G);
                    rec[c][m] = lv.march_div ? precip(d) : qrecip(d);
                }
        }
        __syncthreads();
    }

    // recomputed at each use: held, it would cost eight cells their registers
    __device__ __forceinline__ T diagonal(int c, int m, const T* G) const {
        T d = face_sum(b[c][m]);
        if (kBnd) d = d + G[c * half + min((int)threadIdx.x + m * kBottomThreads, half - 1)];
        return d;
    }

    template <int c>
    __device__ __forceinline__ void colour(T* P, const T* G, T h2) {
#pragma unroll
        for (int m = 0; m < K; ++m) {
            const int e = threadIdx.x + m * kBottomThreads;
            if (e >= half) continue;
            const T d = diagonal(c, m, G);
            T r;
            if constexpr (kRec) r = rec[c][m];
            else r = qrecip(d);                        // FP64: precip is the same
            P[c * half + e] = cell_update(b[c][m], nb[c][m], P + (1 - c) * half, h2, f[c][m], d, r);
        }
        __syncthreads();
    }

    __device__ __forceinline__ void sweeps(T* P, const T* G, T h2, int n) {
        for (int s = 0; s < n; ++s) {
            // keeps the unpacked neighbour offsets (and the diagonals) from
            // being hoisted out of the loop: 64 registers more than there are
#pragma unroll
            for (int m = 0; m < 2 * K; ++m) {
                for (int d = 0; d < 3; ++d) asm volatile("" : "+v"(nb[m / K][m % K][d]));
                asm volatile("" : "+v"(b[m / K][m % K][0]));
            }
            colour<0>(P, G, h2);
            colour<1>(P, G, h2);
        }
    }

    __device__ __forceinline__ void residual(const T* P, const T* G, T* R, T ih2) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int m = 0; m < K; ++m) {
                const int e = threadIdx.x + m * kBottomThreads;
                if (e < half)
                    R[c * half + e] = cell_residual<kBnd>(b[c][m], nb[c][m], P + (1 - c) * half, P[c * half + e],
                                                          f[c][m], kBnd ? G[c * half + e] : T(0), ih2);
            }
        __syncthreads();
    }

    // phi += the coarse value at(I, J, K) of each cell's parent
    template <typename At>
    __device__ __forceinline__ void prolong(const BottomLevel<T>& lv, T* P, At at) {
        const int t = own_thread();
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int m = 0; m < K; ++m) {
                const int e = t + m * kBottomThreads;
                if (e >= half) continue;
                int ih, j, k, r;
                small_divmod(e, lv.nx >> 1, r, ih);
                small_divmod(r, lv.ny, k, j);
                P[c * half + e] = P[c * half + e] + at(ih, j >> 1, k >> 1);
            }
        __syncthreads();
    }

    __device__ __forceinline__ void write(const BottomLevel<T>& lv, const T* P, T* out) {
        const int nx = lv.nx, hx = nx >> 1, t = own_thread();
#pragma unroll
        for (int m = 0; m < K; ++m) {
            const int e = t + m * kBottomThreads;
            if (e >= half) continue;
            int ih, j, k, r;
            small_divmod(e, hx, r, ih);
            small_divmod(r, lv.ny, k, j);
            const int s = (j + k) & 1;                 // the pair's even cell is red where j + k is even
            out[r * nx + 2 * ih] = P[s * half + e];
            out[r * nx + 2 * ih + 1] = P[(1 - s) * half + e];
        }
    }
};

// The second level's cells (at most 512: one of each colour per thread),
// everything but the neighbour numbers in LDS, by colour; its coefficients
// are fetched when the kernel starts, before they are needed.
template <typename T>
struct SecondLds {
    static constexpr int N = kBottomCells / 8;
    T b[6][N], rec[N], dg[N], f[N], P[N], R[N];
};

template <typename T, bool kBnd>
struct Second {
    unsigned nb[2][3];
    int half;

    __device__ __forceinline__ void load(const BottomLevel<T>& lv, SecondLds<T>& L) {
        half = (lv.nx >> 1) * lv.ny * lv.nz;
        const int e = threadIdx.x;
        for (int c = 0; c < 2; ++c) {
            const CellAt q = cell_at(lv, c, min(e, half - 1));
            for (int d = 0; d < 3; ++d) nb[c][d] = q.nb[d];
            if (e >= half) continue;
            T b[6];
            cell_coeffs(lv, q, b);
            T d = face_sum(b);
            if (kBnd) {
                const T g = bnd_diag(lv.bnd, q.i, q.j, q.k, lv.nx, lv.ny, lv.nz);
                L.dg[c * half + e] = g;
                d = d + g;
            }
            for (int k = 0; k < 6; ++k) L.b[k][c * half + e] = b[k];
            L.rec[c * half + e] = lv.march_div ? precip(d) : qrecip(d);
            L.P[c * half + e] = T(0);
        }
    }

    __device__ __forceinline__ void sweeps(SecondLds<T>& L, T h2, int n) {
        const int e = threadIdx.x;
        for (int s = 0; s < 2 * n; ++s) {
            const int c = s & 1, o = c * half + e;
            if (e < half) {
                T b[6];
                for (int k = 0; k < 6; ++k) b[k] = L.b[k][o];
                T d = face_sum(b);
                if (kBnd) d = d + L.dg[o];
                const unsigned n3[3] = {c ? nb[1][0] : nb[0][0], c ? nb[1][1] : nb[0][1], c ? nb[1][2] : nb[0][2]};
                L.P[o] = cell_update(b, n3, L.P + (1 - c) * half, h2, L.f[o], d, L.rec[o]);
            }
            __syncthreads();
        }
    }

    __device__ __forceinline__ void residual(SecondLds<T>& L, T ih2) {
        const int e = threadIdx.x;
        if (e < half)
            for (int c = 0; c < 2; ++c) {
                const int o = c * half + e;
                T b[6];
                for (int k = 0; k < 6; ++k) b[k] = L.b[k][o];
                L.R[o] = cell_residual<kBnd>(b, nb[c], L.P + (1 - c) * half, L.P[o], L.f[o], kBnd ? L.dg[o] : T(0), ih2);
            }
        __syncthreads();
    }
};

// F_c = the mean of the 8 children's residuals (x fastest, then y, then z);
// at most 512 coarse cells, one per thread, to at(I, J, K).
template <typename T, typename At>
__device__ __forceinline__ void bottom_restrict(const BottomLevel<T>& lv, const T* R, At at) {
    const int cx = lv.nx >> 1, cy = lv.ny >> 1, cz = lv.nz >> 1, half = cx * lv.ny * lv.nz;
    const int e = threadIdx.x;
    if (e < cx * cy * cz) {
        int I, J, K, r;
        small_divmod(e, cx, r, I);
        small_divmod(r, cy, K, J);
        T s = T(0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int di = q & 1, dj = (q >> 1) & 1, dk = q >> 2;
            s = s + R[((di + dj + dk) & 1) * half + ((2 * K + dk) * lv.ny + 2 * J + dj) * cx + I];
        }
        at(I, J, K) = T(0.125) * s;
    }
    __syncthreads();
}

template <typename T, int K, bool kBnd>
__device__ __forceinline__ void bottom_body(const BottomArgs<T>& A) {
    constexpr int N0 = 2 * K * kBottomThreads, Nc = kBottomCells / 8;
    __shared__ T P0[N0], G0[kBnd ? N0 : 1], Fc[Nc], Xc[Nc];
    __shared__ SecondLds<T> L;
    __shared__ double work[kMatvecParts * kCoarseMax];  // residuals of the first level, or the coarsest solve's sums
    __shared__ double rhs[kCoarseMax], x[kCoarseMax], mean;
    static_assert(sizeof(work) >= sizeof(P0), "the first level's residuals use the same LDS");
    T* const R0 = reinterpret_cast<T*>(work);
    const BottomLevel<T>&l0 = A.lev[0], &l1 = A.lev[1];
    const bool two = A.nlev > 2;                        // a second smoothed level between
    Owned<T, K, kBnd> a;
    Second<T, kBnd> o;
    if (two) o.load(l1, L);
    a.load(l0, A.f, P0, G0);
    const int cx = l1.nx >> (two ? 1 : 0), cy = l1.ny >> (two ? 1 : 0), nc = cx * cy * (l1.nz >> (two ? 1 : 0));
    const int hx1 = l1.nx >> 1, ny1 = l1.ny, half1 = hx1 * l1.ny * l1.nz;
    auto coarse = [&](T* p) { return [=](int I, int J, int Kz) -> T& { return p[(Kz * cy + J) * cx + I]; }; };
    auto second = [&](T* p) {
        return [=](int I, int J, int Kz) -> T& {
            return p[((I + J + Kz) & 1) * half1 + (Kz * ny1 + J) * hx1 + (I >> 1)];
        };
    };
    for (int visit = 0; visit < 2; ++visit) {
        if (visit) {
            if (two) a.prolong(l0, P0, second(L.P));
            else a.prolong(l0, P0, coarse(Xc));
        }
        a.sweeps(P0, G0, l0.h2, visit ? A.post : A.pre);
        if (visit) break;
        a.residual(P0, G0, R0, T(1) / l0.h2);
        if (two) {
            bottom_restrict(l0, R0, second(L.f));
            o.sweeps(L, l1.h2, A.pre);
            o.residual(L, T(1) / l1.h2);
            bottom_restrict(l1, L.R, coarse(Fc));
        } else {
            bottom_restrict(l0, R0, coarse(Fc));
        }
        b_coarse<T, kBottomThreads>(nc, A.singular, A.minv, Fc, Xc, rhs, x, work, &mean);
        if (two) {
            const int e = threadIdx.x;
            if (e < half1) {
                int ih, j, k, r;
                small_divmod(e, hx1, r, ih);
                small_divmod(r, ny1, k, j);
                for (int c = 0; c < 2; ++c)
                    L.P[c * half1 + e] = L.P[c * half1 + e] + Xc[((k >> 1) * cy + (j >> 1)) * cx + ih];
            }
            __syncthreads();
            o.sweeps(L, l1.h2, A.post);
        }
    }
    a.write(l0, P0, A.phi);
}

template <typename T, int K, bool kBnd>
__global__ __launch_bounds__(kBottomThreads) void k_bottom(BottomArgs<T> a) {
    bottom_body<T, K, kBnd>(a);
}

template <typename T, int K>
__global__ __launch_bounds__(kBottomThreads) void k_bottom_multi(const BottomArgs<T>* __restrict__ descs) {
    bottom_body<T, K, false>(descs[blockIdx.x]);        // batches have no outflow sides
}

template <typename T, int K>
void launch_form(const BottomArgs<T>& a, hipStream_t st) {
    if (a.lev[0].has_bnd) hipLaunchKernelGGL((k_bottom<T, K, true>), dim3(1), dim3(kBottomThreads), 0, st, a);
    else hipLaunchKernelGGL((k_bottom<T, K, false>), dim3(1), dim3(kBottomThreads), 0, st, a);
}

}  // namespace

template <typename T>
hipError_t launch_bottom(const BottomArgs<T>& a, hipStream_t st) {
    const int n = bottom_cells(a);
    if (n > kBottomCells || a.nlev < 2 || a.nlev > kMaxBottomLevels) return hipErrorInvalidValue;
    if (n > 4 * kBottomThreads) launch_form<T, 4>(a, st);
    else if (n > 2 * kBottomThreads) launch_form<T, 2>(a, st);
    else launch_form<T, 1>(a, st);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_bottom_multi(const BottomArgs<T>* d, int nprob, int cells, hipStream_t st) {
    if (nprob <= 0) return hipSuccess;
    if (cells < 1 || cells > kBottomCells) return hipErrorInvalidValue;
    const dim3 nt(kBottomThreads);
    if (cells > 4 * kBottomThreads) hipLaunchKernelGGL((k_bottom_multi<T, 4>), dim3(nprob), nt, 0, st, d);
    else if (cells > 2 * kBottomThreads) hipLaunchKernelGGL((k_bottom_multi<T, 2>), dim3(nprob), nt, 0, st, d);
    else hipLaunchKernelGGL((k_bottom_multi<T, 1>), dim3(nprob), nt, 0, st, d);
    return hipGetLastError();
}

template hipError_t launch_bottom<double>(const BottomArgs<double>&, hipStream_t);
template hipError_t launch_bottom<float>(const BottomArgs<float>&, hipStream_t);
template hipError_t launch_bottom_multi<double>(const BottomArgs<double>*, int, int, hipStream_t);
template hipError_t launch_bottom_multi<float>(const BottomArgs<float>*, int, int, hipStream_t);

}  // namespace mg
