// Nodal (cell-velocity) projection for gfx950: phi on the cell corners,
// cell-centred velocities, the same divergence constraint as the MAC
// projection (arXiv:1910.12979, Sec. 2), solved by multigrid (Sec. 3).
//
// Discretisation: trilinear elements on the nodes with a cell-constant
// coefficient sigma = beta0 / rho.  Divided by the node volume h^3,
//   (L phi)_n = 1/(12 h^2) sum_{cells c at n} sigma_c
//               [ sum of phi over the 4 corners of c across a face or the body
//                 diagonal from n  -  4 phi_n ]
// (corners joined to n by an edge have weight 0 in the element stiffness),
//   f_n = 1/(4h) sum_c beta0_c (+-u_c +- v_c +- w_c) - 1/8 sum_c beta0_c S_c
// (+ for a cell on the high side of n in that direction), and the cells'
// velocities are corrected by their mean gradient of phi over rho.  A solid
// wall is a natural boundary (its nodes are unknowns, only existing cells
// contribute); in a periodic direction node n is node 0.
//
// Multigrid: four-colour Gauss-Seidel, colour (J mod 2) + 2 (K mod 2) in the
// order 0..3 (coupled nodes differ by one in at least two coordinates, so in J
// or K, and their colours differ; each x-row has one colour); residual, full-weighting
// restriction 1/8 sum_d prod(1 - |d_i|/2) r_{2C+d}; trilinear prolongation;
// coarse sigma the mean of the 8 fine cells; exact coarsest solve (at most
// 512 nodes) by the dense inverse of -A + c 1 1^T.  Every per-node
// expression is evaluated in one fixed order, without FMA contraction beyond
// the multiply-adds written out (nodal_march.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstring>
#include <utility>
#include <vector>
#include <new>
#include <string>

#include "dense.h"
#include "devmath.h"
#include "mg_internal.h"
#include "nodal_march.h"
#include "runtime.h"

namespace mg {
namespace {

constexpr int kNodBlock = 256;

__device__ inline int nod_cell(int I, int s, int n, int per) {
    int c = s ? I : I - 1;
    if (per) return c < 0 ? c + n : (c >= n ? c - n : c);
    return (c >= 0 && c < n) ? c : -1;
}

__device__ inline int nod_node(int I, int o, int N, int per) {
    int m = I + o;
    if (per) return m < 0 ? m + N : (m >= N ? m - N : m);
    return (m >= 0 && m < N) ? m : -1;
}

template <typename T>
__device__ inline size_t nidx(const NodLevelT<T>& L, int I, int J, int K) {
    return ((size_t)K * L.Ny + J) * L.Nx + I;
}

template <typename T>
__device__ inline size_t cidx3(const NodLevelT<T>& L, int i, int j, int k) {
    return ((size_t)k * L.ny + j) * L.nx + i;
}

// Neighbour and cell indices of node coordinate X along one direction:
// nodes X-1 / X+1 (m[0], m[1]) and the cells on its low / high side (c[0],
// c[1], e[s] = whether that cell exists).
struct NodAxis {
    int m[2], c[2];
    bool e[2];
};

__device__ inline NodAxis nod_axis(int X, int N, int n, int per) {
    NodAxis a;
    if (per) {
        a.m[0] = X > 0 ? X - 1 : N - 1;
        a.m[1] = X + 1 < N ? X + 1 : 0;
        a.c[0] = X > 0 ? X - 1 : n - 1;
        a.c[1] = X;
        a.e[0] = a.e[1] = true;
    } else {
        a.m[0] = X - 1;
        a.m[1] = X + 1;
        a.c[0] = X - 1;
        a.c[1] = X;
        a.e[0] = X >= 1;
        a.e[1] = X < n;
    }
    return a;
}

// The 20 neighbours of node (I, J, K) that the stencil couples (moved in at
// least two directions), each loaded once: v[dz+1][dy+1][dx+1]; entries
// whose node does not exist (beyond a wall) are never used and stay 0.
template <typename T>
struct NodNbr {
    T v[3][3][3];
};

template <typename T>
__device__ inline void nod_load_nbrs(const NodLevelT<T>& L, const T* __restrict__ phi, int I, const NodAxis& ax,
                                     const NodAxis& ay, const NodAxis& az, int J, int K, NodNbr<T>& N) {
    const long long Nx = L.Nx, NxNy = (long long)L.Nx * L.Ny;
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
            for (int dx = -1; dx <= 1; ++dx) {
                if ((dx != 0) + (dy != 0) + (dz != 0) < 2) continue;
                const bool ok = (dx == 0 || ax.e[dx > 0]) && (dy == 0 || ay.e[dy > 0]) && (dz == 0 || az.e[dz > 0]);
                const long long xi = dx == 0 ? I : ax.m[dx > 0];
                const long long yi = dy == 0 ? J : ay.m[dy > 0];
                const long long zi = dz == 0 ? K : az.m[dz > 0];
                N.v[dz + 1][dy + 1][dx + 1] = ok ? phi[zi * NxNy + yi * Nx + xi] : T(0);
            }
}

// num = sum_c sigma_c sum_{4 far corners} phi, den = 4 sum_c sigma_c over
// the existing cells at node (I, J, K), in the oracle's order (cells sz, sy,
// sx; far corners of the cell on side (sx, sy, sz): x+y, x+z, y+z, x+y+z
// moved), with per-axis index tables and each neighbour loaded once.
template <typename T>
__device__ inline void nod_stencil_fast(const NodLevelT<T>& L, const T* __restrict__ phi, int I, int J, int K,
                                        T& num, T& den) {
    const NodAxis ax = nod_axis(I, L.Nx, L.nx, L.px);
    const NodAxis ay = nod_axis(J, L.Ny, L.ny, L.py);
    const NodAxis az = nod_axis(K, L.Nz, L.nz, L.pz);
    NodNbr<T> N;
    nod_load_nbrs(L, phi, I, ax, ay, az, J, K, N);
    const long long nx = L.nx, nxny = (long long)L.nx * L.ny;
    num = T(0);
    den = T(0);
#pragma unroll
    for (int sz = 0; sz < 2; ++sz) {
        if (!az.e[sz]) continue;
        const int oz = sz ? 2 : 0;
#pragma unroll
        for (int sy = 0; sy < 2; ++sy) {
            if (!ay.e[sy]) continue;
            const int oy = sy ? 2 : 0;
#pragma unroll
            for (int sx = 0; sx < 2; ++sx) {
                if (!ax.e[sx]) continue;
                const int ox = sx ? 2 : 0;
                const T sig = L.sig[az.c[sz] * nxny + ay.c[sy] * nx + ax.c[sx]];
                T acc = T(0);
                acc += N.v[1][oy][ox];
                acc += N.v[oz][1][ox];
                acc += N.v[oz][oy][1];
                acc += N.v[oz][oy][ox];
                num += sig * acc;
                den += T(4) * sig;
            }
        }
    }
}

// Point loops of the reductions: 64 x 4 threads per workgroup over (x, y),
// the workgroups of a launch striding over x, y and the planes; no
// per-thread index division.  The partial row of a workgroup is its flat
// index.
constexpr int kPtX = 64, kPtY = 4;
__device__ inline int part_row() { return (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x; }

// sigma = beta0 / rho per cell; partial rows {0, 0, bad, #non-finite} of
// rho and beta0 (256^3 nodes 155 us while it also read S and the velocities for
// their checks, which the right-hand side now makes).
__global__ __launch_bounds__(kNodBlock) void k_nod_sigma(NodLevel L, const double* __restrict__ rho,
                                                         const double* __restrict__ b0c,
                                                         double* __restrict__ partials) {
    double bad = 0.0, nonfin = 0.0;
    for (int k = blockIdx.z; k < L.nz; k += gridDim.z)
    for (int j = blockIdx.y * kPtY + threadIdx.y; j < L.ny; j += gridDim.y * kPtY)
    for (int i = blockIdx.x * kPtX + threadIdx.x; i < L.nx; i += gridDim.x * kPtX) {
        const size_t c = cidx3(L, i, j, k);
        const double r = rho[c], b = b0c[k];
        if (!isfinite(r) || !isfinite(b)) nonfin += 1.0;
        if (!(r > 0.0) || !(b > 0.0)) bad = 1.0;
        L.sig[c] = b / r;
    }
    reduce_row256(0.0, 0.0, bad, nonfin, partials + (size_t)part_row() * kReduceWidth);
}

// f_n and partial rows {sum f, sum |f|, 0, #non-finite of u, v, w, S}.  A
// wavefront marches up through a chunk of planes with 64 columns of four rows:
// a cell layer's sums over the four cells around a node are formed once, from
// the lane's own column and the one of the lane below, and serve the planes
// below and above it.  Bound by reading u, v, w and S once: 256^3 nodes 177 us
// (3.8 TB/s; 407 us with a node gathering its eight cells).
constexpr int kRhsTX = 63;
__global__ __launch_bounds__(64 * kNodResidWaves) void k_nod_rhs(NodLevel L, const double* __restrict__ b0c,
                                                                const double* __restrict__ u,
                                                                const double* __restrict__ v,
                                                                const double* __restrict__ w,
                                                                const double* __restrict__ S, int tz, int ntx,
                                                                int nty, double* __restrict__ partials) {
    constexpr int R = kNodResidRows;
    static_assert(64 * kNodResidWaves == kNodBlock, "reduce_row256");
    const int tile = xcd_order(blockIdx.x, gridDim.x);
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tc = tile / (ntx * nty);
    const int wx = threadIdx.x;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int gI = tx * kRhsTX - 1 + wx, gJ = (ty * kNodResidWaves + p) * R;
    const int Ka = tc * tz, Kb = min(Ka + tz, L.Nz);
    auto in = [](int g, int n, int per) { return per || (g >= 0 && g < n); };
    const bool xc = in(gI, L.nx, L.px);
    const size_t nxny = (size_t)L.nx * L.ny;
    size_t row[R + 1];                            // cell rows gJ - 1 .. gJ + 3
    bool ok[R + 1];
#pragma unroll
    for (int j = 0; j <= R; ++j) {
        row[j] = (size_t)fold(gJ - 1 + j, L.ny, L.py) * L.nx + fold(gI, L.nx, L.px);
        ok[j] = xc && in(gJ - 1 + j, L.ny, L.py);
    }
    double sf = 0.0, saf = 0.0, nonfin = 0.0;
    const double h4 = 4.0 * L.h;
    // beta0-weighted sums over a layer's cells around the nodes: of +-u +- v, of w, of S
    struct Layer {
        double a[R], w[R], s[R];
    };
    auto layer = [&](int k, Layer& y) {
        const bool zk = in(k, L.nz, L.pz);
        const int kf = fold(k, L.nz, L.pz);
        const size_t o = (size_t)kf * nxny;
        double qu[R + 1], qv[R + 1], qw[R + 1], qs[R + 1];
#pragma unroll
        for (int j = 0; j <= R; ++j) {
            qu[j] = u[o + row[j]];
            qv[j] = v[o + row[j]];
            qw[j] = w[o + row[j]];
            qs[j] = S[o + row[j]];
        }
        const double b = b0c[kf];
#pragma unroll
        for (int j = 0; j <= R; ++j) {
            const bool e = ok[j] && zk;
            if (!isfinite(qu[j]) || !isfinite(qv[j]) || !isfinite(qw[j]) || !isfinite(qs[j])) nonfin += 1.0;
            qu[j] = e ? qu[j] : 0.0;
            qv[j] = e ? qv[j] : 0.0;
            qw[j] = e ? qw[j] : 0.0;
            qs[j] = e ? qs[j] : 0.0;
            qu[j] = qu[j] - lane_lo(qu[j]);
            qv[j] = qv[j] + lane_lo(qv[j]);
            qw[j] = qw[j] + lane_lo(qw[j]);
            qs[j] = qs[j] + lane_lo(qs[j]);
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            y.a[j] = b * ((qu[j] + qu[j + 1]) + (qv[j + 1] - qv[j]));
            y.w[j] = b * (qw[j] + qw[j + 1]);
            y.s[j] = b * (qs[j] + qs[j + 1]);
        }
    };
    Layer lo, hi;
    layer(Ka - 1, lo);
    for (int K = Ka; K < Kb; ++K) {
        layer(K, hi);
        const bool own = wx >= 1 && gI < L.Nx;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (own && gJ + j < L.Ny) {
                const double fn = ((lo.a[j] + hi.a[j]) + (hi.w[j] - lo.w[j])) / h4 - 0.125 * (lo.s[j] + hi.s[j]);
                L.f[nidx(L, gI, gJ + j, K)] = fn;
                sf += fn;
                saf += fabs(fn);
            }
        }
        lo = hi;
    }
    reduce_row256(sf, saf, 0.0, nonfin, partials + (size_t)blockIdx.x * kReduceWidth);
}

// One colour of the Gauss-Seidel sweep; thread (I, tj, tk) owns node
// (I, 2 tj + (col & 1), 2 tk + (col >> 1)).
template <typename T>
__global__ void k_nod_gs(NodLevelT<T> L, int col) {
    const int I = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    const int J = 2 * (int)(blockIdx.y * blockDim.y + threadIdx.y) + (col & 1);
    const int K = 2 * (int)(blockIdx.z * blockDim.z + threadIdx.z) + (col >> 1);
    if (I >= L.Nx || J >= L.Ny || K >= L.Nz) return;
    T num, den;
    nod_stencil_fast(L, L.phi, I, J, K, num, den);
    const size_t n = nidx(L, I, J, K);
    const T c12 = (T)(12.0 * (L.h * L.h));
    L.phi[n] = pdiv(num - c12 * L.f[n], den);
}

// r = f - L phi at node (I, J, K): cells sz, sy, sx, far corners x+y, x+z,
// y+z, x+y+z of each.
template <typename T>
__device__ inline T nod_resid_at(const NodLevelT<T>& L, int I, int J, int K) {
    const NodAxis ax = nod_axis(I, L.Nx, L.nx, L.px);
    const NodAxis ay = nod_axis(J, L.Ny, L.ny, L.py);
    const NodAxis az = nod_axis(K, L.Nz, L.nz, L.pz);
    NodNbr<T> N;
    nod_load_nbrs(L, L.phi, I, ax, ay, az, J, K, N);
    const size_t n = nidx(L, I, J, K);
    const T pn = L.phi[n];
    T sum = T(0);
    for (int sz = 0; sz < 2; ++sz)
        for (int sy = 0; sy < 2; ++sy)
            for (int sx = 0; sx < 2; ++sx) {
                if (!az.e[sz] || !ay.e[sy] || !ax.e[sx]) continue;
                const int oz = 2 * sz, oy = 2 * sy, ox = 2 * sx;
                const T sig = L.sig[cidx3(L, ax.c[sx], ay.c[sy], az.c[sz])];
                T acc = T(0);
                acc += N.v[1][oy][ox];
                acc += N.v[oz][1][ox];
                acc += N.v[oz][oy][1];
                acc += N.v[oz][oy][ox];
                sum += sig * (acc - T(4) * pn);
            }
    return L.f[n] - pdiv(sum, (T)(12.0 * L.h * L.h));
}

// Restricted residual of a level of the bottom kernel launched by itself: the
// bottom kernel's sums, each coarse node forming the residuals around it.
template <typename T>
__global__ __launch_bounds__(64) void k_nod_restrict_each(NodLevelT<T> F, NodLevelT<T> C) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= (int)C.nodes()) return;
    const int X[3] = {2 * (c % C.Nx), 2 * (c / C.Nx % C.Ny), 2 * (c / (C.Nx * C.Ny))};
    const int Nn[3] = {F.Nx, F.Ny, F.Nz}, per[3] = {F.px, F.py, F.pz};
    T s = T(0);
    for (int d = 0; d < 27; ++d) {
        const int D[3] = {d % 3 - 1, d / 3 % 3 - 1, d / 9 - 1};
        int m[3];
        bool ok = true;
        T w = T(1);
        for (int i = 0; i < 3; ++i) {
            m[i] = nod_node(X[i], D[i], Nn[i], per[i]);
            if (m[i] < 0) ok = false;
            if (D[i] != 0) w *= T(0.5);
        }
        if (ok) s += w * nod_resid_at(F, m[0], m[1], m[2]);
    }
    C.f[c] = T(0.125) * s;
    C.phi[c] = T(0);
}

// fine phi += trilinear interpolation of the coarse phi.  One thread per
// coarse node (I, J, K) updates the up to 8 fine nodes (2I + dx, 2J + dy,
// 2K + dz), dx, dy, dz in {0, 1}, from the 8 coarse values around it,
// loaded once; per fine node the parents are summed in the order (z, y, x)
// with the weight 1 or 1/2 per direction.
template <typename T>
__global__ void k_nod_prolong(NodLevelT<T> F, NodLevelT<T> C) {
    const int I = blockIdx.x * blockDim.x + threadIdx.x;
    const int J = blockIdx.y * blockDim.y + threadIdx.y;
    const int K = blockIdx.z * blockDim.z + threadIdx.z;
    if (I >= C.Nx || J >= C.Ny || K >= C.Nz) return;
    // coarse node + 1 in each direction (the periodic image; beyond a wall
    // the node itself, whose value is never used: no fine node lies there)
    const int I1 = I + 1 < C.Nx ? I + 1 : (C.px ? 0 : I);
    const int J1 = J + 1 < C.Ny ? J + 1 : (C.py ? 0 : J);
    const int K1 = K + 1 < C.Nz ? K + 1 : (C.pz ? 0 : K);
    T c[2][2][2];
    c[0][0][0] = C.phi[nidx(C, I, J, K)];
    c[0][0][1] = C.phi[nidx(C, I1, J, K)];
    c[0][1][0] = C.phi[nidx(C, I, J1, K)];
    c[0][1][1] = C.phi[nidx(C, I1, J1, K)];
    c[1][0][0] = C.phi[nidx(C, I, J, K1)];
    c[1][0][1] = C.phi[nidx(C, I1, J, K1)];
    c[1][1][0] = C.phi[nidx(C, I, J1, K1)];
    c[1][1][1] = C.phi[nidx(C, I1, J1, K1)];
#pragma unroll
    for (int dz = 0; dz < 2; ++dz)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx) {
                const int X = 2 * I + dx, Y = 2 * J + dy, Z = 2 * K + dz;
                if (X >= F.Nx || Y >= F.Ny || Z >= F.Nz) continue;
                const int D[3] = {dx, dy, dz};
                T v = T(0);
#pragma unroll
                for (int bz = 0; bz < 2; ++bz)
#pragma unroll
                    for (int by = 0; by < 2; ++by)
#pragma unroll
                        for (int bx = 0; bx < 2; ++bx) {
                            const int B[3] = {bx, by, bz};
                            bool ok = true;
                            T w = T(1);
#pragma unroll
                            for (int d = 0; d < 3; ++d) {
                                if (D[d] == 0) {
                                    if (B[d]) ok = false;    // an even fine index has one parent
                                } else {
                                    w *= T(0.5);
                                }
                            }
                            if (ok) v += w * c[bz][by][bx];
                        }
                const size_t n = nidx(F, X, Y, Z);
                F.phi[n] = F.phi[n] + v;
            }
}

__global__ void k_nod_avg_sigma(NodLevel F, NodLevel C) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i >= C.nx || j >= C.ny || k >= C.nz) return;
    double s = 0.0;
    for (int dk = 0; dk < 2; ++dk)
        for (int dj = 0; dj < 2; ++dj)
            for (int di = 0; di < 2; ++di) s += F.sig[cidx3(F, 2 * i + di, 2 * j + dj, 2 * k + dk)];
    C.sig[cidx3(C, i, j, k)] = 0.125 * s;
}

// Coarsest level: M = -A + c 1 1^T (c the mean diagonal), inverted (dense.h).
// Row n of -A: -(1/(12 h^2)) sum_c sigma_c (far corners - 4 e_n).  Entry e of
// the 20 off-diagonal ones: 0..11 the nodes moved in two directions (the
// cells on both sides of the plane they lie in), 12..19 the body diagonals.
struct NodCoarseRows {
    NodLevel L;
    double s12;
    __device__ double sigma(int i, int j, int k) const {
        return (i < 0 || j < 0 || k < 0) ? 0.0 : L.sig[cidx3(L, i, j, k)];
    }
    __device__ void operator()(int r, int e, double& val, int& nb) const {
        const int X[3] = {r % L.Nx, (r / L.Nx) % L.Ny, r / (L.Nx * L.Ny)};
        const int Nn[3] = {L.Nx, L.Ny, L.Nz}, nc[3] = {L.nx, L.ny, L.nz}, per[3] = {L.px, L.py, L.pz};
        int side[3], still = 3;                        // side per direction; `still`: the direction not moved in
        if (e < 12) {
            still = e >> 2;
            const int d1 = still == 0 ? 1 : 0, d2 = still == 2 ? 1 : 2;
            side[d1] = e & 1;
            side[d2] = (e >> 1) & 1;
            side[still] = 0;
        } else {
            side[0] = e & 1;
            side[1] = (e >> 1) & 1;
            side[2] = ((e - 12) >> 2) & 1;
        }
        int m[3], c[3];
        bool ok = true;
        for (int d = 0; d < 3; ++d) {
            m[d] = d == still ? X[d] : nod_node(X[d], side[d] ? 1 : -1, Nn[d], per[d]);
            c[d] = nod_cell(X[d], side[d], nc[d], per[d]);
            ok = ok && m[d] >= 0;
        }
        val = 0.0;
        nb = 0;
        if (!ok) return;
        double s = sigma(c[0], c[1], c[2]);
        if (still < 3) {
            c[still] = nod_cell(X[still], 1, nc[still], per[still]);
            s += sigma(c[0], c[1], c[2]);
        }
        val = s * s12;
        nb = (int)nidx(L, m[0], m[1], m[2]);
    }
    __device__ double diag(int r) const {
        const int X[3] = {r % L.Nx, (r / L.Nx) % L.Ny, r / (L.Nx * L.Ny)};
        const int nc[3] = {L.nx, L.ny, L.nz}, per[3] = {L.px, L.py, L.pz};
        double d = 0.0;
        for (int q = 0; q < 8; ++q)
            d += sigma(nod_cell(X[0], q & 1, nc[0], per[0]), nod_cell(X[1], (q >> 1) & 1, nc[1], per[1]),
                       nod_cell(X[2], q >> 2, nc[2], per[2]));
        return 4.0 * d * s12;
    }
};

__global__ __launch_bounds__(kDenseThreads) void k_nod_coarse_setup(NodCoarseRows R, double* __restrict__ M) {
    __shared__ DenseLds<20> S;
    dense_invert<20>((int)R.L.nodes(), 1, M, S, R, [&](int r) { return R.diag(r); });
}

__global__ __launch_bounds__(256) void k_nod_coarse_build(NodCoarseRows R, double* __restrict__ M) {
    dense_build_row<20>((int)R.L.nodes(), 1, M, R, [&](int r) { return R.diag(r); });
}

hipError_t launch_nod_coarse_setup(const NodLevel& L, double* minv, double* scratch, hipStream_t st) {
    if (L.nodes() < 1 || L.nodes() > (size_t)kCoarseMax) return hipErrorInvalidValue;
    const NodCoarseRows R{L, 1.0 / (12.0 * L.h * L.h)};
    const int n = (int)L.nodes();
    if (n <= kDenseReg) {
        hipLaunchKernelGGL(k_nod_coarse_setup, dim3(1), dim3(kDenseThreads), 0, st, R, minv);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_nod_coarse_build, dim3(n), dim3(256), 0, st, R, minv);
    return launch_dense_blocks(minv, n, scratch, st);
}

// U_c -= (G phi)_c / rho_c with phi - mean (mean = *phi_sum / nodes); phi_out
// (nullable) = phi - mean at the nodes (written by the threads of the first
// nodes).
__global__ void k_nod_correct(NodLevel L, const double* __restrict__ rho, const double* __restrict__ phi_sum,
                              double* __restrict__ u, double* __restrict__ v, double* __restrict__ w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i >= L.nx || j >= L.ny || k >= L.nz) return;
    const double m = phi_sum[0] / (double)L.nodes();
    const int lo[3] = {i, j, k};
    const int Nn[3] = {L.Nx, L.Ny, L.Nz}, per[3] = {L.px, L.py, L.pz};
    int hi[3];
    for (int d = 0; d < 3; ++d) hi[d] = nod_node(lo[d], 1, Nn[d], per[d]);
    auto P = [&](int x, int y, int z) { return L.phi[nidx(L, x, y, z)] - m; };
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) {
            const int y = a ? hi[1] : lo[1], z = b ? hi[2] : lo[2];
            g0 += P(hi[0], y, z) - P(lo[0], y, z);
            const int x = a ? hi[0] : lo[0];
            g1 += P(x, hi[1], z) - P(x, lo[1], z);
            const int yy = b ? hi[1] : lo[1];
            g2 += P(x, yy, hi[2]) - P(x, yy, lo[2]);
        }
    const size_t c = cidx3(L, i, j, k);
    const double h4 = 4.0 * L.h;
    u[c] = u[c] - (g0 / h4) / rho[c];
    v[c] = v[c] - (g1 / h4) / rho[c];
    w[c] = w[c] - (g2 / h4) / rho[c];
}

__global__ void k_nod_shift_out(size_t n, const double* __restrict__ phi, const double* __restrict__ phi_sum,
                                double* __restrict__ out) {
    const double m = phi_sum[0] / (double)n;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
        out[e] = phi[e] - m;
}

// ---------------------------------------------------------------------------
// Bottom of the nodal V-cycle in one workgroup: from the first level that
// fits (with the next coarser ones) in LDS down to the coarsest solve and
// back, with barriers between dependent steps instead of one launch of a few
// microseconds per colour, residual, restriction and prolongation.  Per node
// the arithmetic is that of the per-level kernels (the same sums in the same
// order; a cell beyond a wall adds an exact zero where they leave it out), so
// a bottom launch gives the same bits as the launches it replaces.
//
// phi, the residual and sigma are in LDS, sigma inside a border that holds
// the periodic images or zeros beyond walls, so that a node's eight cells are
// at fixed offsets; a thread owns the same nodes of each colour throughout
// and keeps their right-hand sides and coordinates in registers.  What bounds
// a colour phase is then the 28 LDS reads and 56 operations of an update
// (sigma from global memory and 64-bit index arithmetic before: from 16 x 16 x
// 17 nodes down 126 -> 69 us in FP64, from 24 x 16 x 21 175 -> 78 us in FP32).
// ---------------------------------------------------------------------------
constexpr int kNodBottomThreads = 1024;

// Capacities: nodes and bordered cells of the first and second level, nodes
// of each colour a thread owns, coarsest nodes below a second level (a level
// directly above the coarsest may have up to kCoarseMax there).
template <typename T>
struct NodBottomCap {
    static constexpr int f = sizeof(T) == 8 ? 1 : 2;
    static constexpr int nodes = 5120 * f, cells = 5888 * f, nodes1 = 768 * f, cells1 = 1024 * f;
    static constexpr int own = sizeof(T) == 8 ? 2 : 3, own1 = 1, coarse = 160;
};

template <typename T>
struct NodBottomArgs {
    int nlev;                           // bottom levels, 2 or 3; the last one is solved directly
    NodLevelT<T> lev[3];                // sig global; phi, f of lev[0] global (in and out)
    const double* minv;
    int pre, post;
};

inline __host__ __device__ int nod_bordered(const int N[3]) { return (N[0] + 1) * (N[1] + 1) * (N[2] + 1); }
inline int nod_colour_max(int Nx, int Ny, int Nz) { return Nx * ((Ny + 1) / 2) * ((Nz + 1) / 2); }

// sigma of L into the bordered array S: entry (x, y, z) is cell (x - 1, y - 1, z - 1).
template <typename T>
__device__ __forceinline__ void nb_load_sigma(const NodLevelT<T>& L, T* S) {
    const int bx = L.Nx + 1, by = L.Ny + 1, n = bx * by * (L.Nz + 1);
    for (int e = threadIdx.x; e < n; e += kNodBottomThreads) {
        int x, y, z, r;
        small_divmod(e, bx, r, x);
        small_divmod(r, by, z, y);
        const int i = nod_cell(x, 0, L.nx, L.px), j = nod_cell(y, 0, L.ny, L.py), k = nod_cell(z, 0, L.nz, L.pz);
        S[e] = (i < 0 || j < 0 || k < 0) ? T(0) : L.sig[(k * L.ny + j) * L.nx + i];
    }
}

// Coordinates of node e of colour col (10 bits each), or -1 past the last.
template <typename T>
__device__ __forceinline__ int nb_own(const NodLevelT<T>& L, int col, int e) {
    const int hy = (L.Ny + 1 - (col & 1)) >> 1, hz = (L.Nz + 1 - (col >> 1)) >> 1;
    if (e >= L.Nx * hy * hz) return -1;
    int I, r, jh, kh;
    small_divmod(e, L.Nx, r, I);
    small_divmod(r, hy, kh, jh);
    return I | (2 * jh + (col & 1)) << 10 | (2 * kh + (col >> 1)) << 20;
}

// The neighbourhood of a node: v[dz][dy][dx] for the 20 coupled nodes (beyond
// a wall some existing node, whose cells' sigma is 0) and its 8 cells.
template <typename T>
struct NbNode {
    T v[3][3][3], s[2][2][2];
    int n;
    __device__ __forceinline__ NbNode(const NodLevelT<T>& L, const T* P, const T* S, int ijk) {
        const int I = ijk & 1023, J = (ijk >> 10) & 1023, K = ijk >> 20;
        auto low = [](int X, int N, int per) { return X > 0 ? X - 1 : (per ? N - 1 : 0); };
        auto high = [](int X, int N, int per) { return X + 1 < N ? X + 1 : (per ? 0 : X); };
        const int x[3] = {low(I, L.Nx, L.px), I, high(I, L.Nx, L.px)};
        const int y[3] = {low(J, L.Ny, L.py) * L.Nx, J * L.Nx, high(J, L.Ny, L.py) * L.Nx};
        const int zs = L.Nx * L.Ny;
        const int z[3] = {low(K, L.Nz, L.pz) * zs, K * zs, high(K, L.Nz, L.pz) * zs};
        n = z[1] + y[1] + I;
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    if ((dx != 1) + (dy != 1) + (dz != 1) >= 2) v[dz][dy][dx] = P[z[dz] + y[dy] + x[dx]];
        const T* c = S + ((K * (L.Ny + 1)) + J) * (L.Nx + 1) + I;
#pragma unroll
        for (int sz = 0; sz < 2; ++sz)
#pragma unroll
            for (int sy = 0; sy < 2; ++sy)
#pragma unroll
                for (int sx = 0; sx < 2; ++sx) s[sz][sy][sx] = c[(sz * (L.Ny + 1) + sy) * (L.Nx + 1) + sx];
    }
    // sum of phi over the four corners of cell (sx, sy, sz) across a face or the diagonal
    __device__ __forceinline__ T far(int sz, int sy, int sx) const {
        T a = v[1][2 * sy][2 * sx];
        a = a + v[2 * sz][1][2 * sx];
        a = a + v[2 * sz][2 * sy][1];
        return a + v[2 * sz][2 * sy][2 * sx];
    }
};

template <typename T>
__device__ __forceinline__ void nb_update(const NodLevelT<T>& L, T* P, const T* S, int ijk, T f) {
    const NbNode<T> q(L, P, S, ijk);
    T num = T(0), den = T(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const T sig = q.s[c >> 2][(c >> 1) & 1][c & 1];
        num = num + sig * q.far(c >> 2, (c >> 1) & 1, c & 1);
        den = den + T(4) * sig;
    }
    P[q.n] = pdiv(num - (T)(12.0 * (L.h * L.h)) * f, den);
}

template <typename T>
__device__ __forceinline__ void nb_residual(const NodLevelT<T>& L, const T* P, const T* S, int ijk, T f, T* R) {
    const NbNode<T> q(L, P, S, ijk);
    const T pn = P[q.n];
    T sum = T(0);
#pragma unroll
    for (int c = 0; c < 8; ++c)
        sum = sum + q.s[c >> 2][(c >> 1) & 1][c & 1] * (q.far(c >> 2, (c >> 1) & 1, c & 1) - T(4) * pn);
    R[q.n] = f - pdiv(sum, (T)(12.0 * L.h * L.h));
}

// A value the compiler cannot see through: what is derived from a node's
// coordinates is then computed at each use, not held for every owned node
// across the sweeps (350 registers more than there are).
__device__ __forceinline__ int at_use(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// A level's nodes as one thread owns them: M of each colour.
template <typename T, int M>
struct NbOwned {
    int ijk[4][M];
    T f[4][M];
    __device__ __forceinline__ void load(const NodLevelT<T>& L) {
#pragma unroll
        for (int q = 0; q < 4 * M; ++q) ijk[q / M][q % M] = nb_own(L, q / M, threadIdx.x + (q % M) * kNodBottomThreads);
    }
    __device__ __forceinline__ void load_f(const NodLevelT<T>& L, const T* F) {
#pragma unroll
        for (int q = 0; q < 4 * M; ++q) {
            const int p = max(ijk[q / M][q % M], 0);
            f[q / M][q % M] = F[((p >> 20) * L.Ny + ((p >> 10) & 1023)) * L.Nx + (p & 1023)];
        }
    }
    __device__ __forceinline__ void sweeps(const NodLevelT<T>& L, T* P, const T* S, int n) {
        for (int s = 0; s < n; ++s) {
#pragma unroll
            for (int col = 0; col < 4; ++col) {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const int p = at_use(ijk[col][m]);
                    if (p >= 0) nb_update(L, P, S, p, f[col][m]);
                }
                __syncthreads();
            }
        }
    }
    __device__ __forceinline__ void residual(const NodLevelT<T>& L, const T* P, const T* S, T* R) {
#pragma unroll
        for (int q = 0; q < 4 * M; ++q) {
            const int p = at_use(ijk[q / M][q % M]);
            if (p >= 0) nb_residual(L, P, S, p, f[q / M][q % M], R);
        }
        __syncthreads();
    }
};

template <typename T>
__device__ void nb_restrict(const NodLevelT<T>& Fl, const T* R, const NodLevelT<T>& Cl, T* cF) {
    const int items = Cl.Nx * Cl.Ny * Cl.Nz;
    const int Nn[3] = {Fl.Nx, Fl.Ny, Fl.Nz}, per[3] = {Fl.px, Fl.py, Fl.pz};
    for (int e = threadIdx.x; e < items; e += kNodBottomThreads) {
        int X[3], r;
        small_divmod(e, Cl.Nx, r, X[0]);
        small_divmod(r, Cl.Ny, X[2], X[1]);
        // fine node 2X - 1 + d of each direction (an existing one beyond a wall, weighted 0)
        int m[3][3];
        T w[3][3];
        const int stride[3] = {1, Fl.Nx, Fl.Nx * Fl.Ny};
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int o = 0; o < 3; ++o) {
                const int g = nod_node(2 * X[d], o - 1, Nn[d], per[d]);
                m[d][o] = max(g, 0) * stride[d];
                w[d][o] = g < 0 ? T(0) : (o == 1 ? T(1) : T(0.5));
            }
        T s = T(0);
#pragma unroll
        for (int q = 0; q < 27; ++q) {
            const int dx = q % 3, dy = (q / 3) % 3, dz = q / 9;
            s = s + (w[0][dx] * w[1][dy] * w[2][dz]) * R[m[2][dz] + m[1][dy] + m[0][dx]];
        }
        cF[e] = T(0.125) * s;
    }
    __syncthreads();
}

template <typename T>
__device__ void nb_prolong(const NodLevelT<T>& Fl, T* P, const NodLevelT<T>& Cl, const T* cP) {
    const int items = Fl.Nx * Fl.Ny * Fl.Nz;
    const int Nc[3] = {Cl.Nx, Cl.Ny, Cl.Nz}, per[3] = {Cl.px, Cl.py, Cl.pz};
    for (int e = threadIdx.x; e < items; e += kNodBottomThreads) {
        int X[3], r;
        small_divmod(e, Fl.Nx, r, X[0]);
        small_divmod(r, Fl.Ny, X[2], X[1]);
        // both coarse parents of each direction (an even index: one, the second weighted 0)
        int m[3][2];
        T w[3][2];
        const int stride[3] = {1, Cl.Nx, Cl.Nx * Cl.Ny};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int lo = X[d] >> 1, odd = X[d] & 1;
            int hi = lo + odd;
            if (per[d] && hi >= Nc[d]) hi -= Nc[d];
            m[d][0] = lo * stride[d];
            m[d][1] = hi * stride[d];
            w[d][0] = odd ? T(0.5) : T(1);
            w[d][1] = odd ? T(0.5) : T(0);
        }
        T v = T(0);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            v = v + (w[0][q & 1] * w[1][(q >> 1) & 1] * w[2][q >> 2]) *
                        cP[m[2][q >> 2] + m[1][(q >> 1) & 1] + m[0][q & 1]];
        P[e] = P[e] + v;
    }
    __syncthreads();
}

template <typename T>
__global__ __launch_bounds__(kNodBottomThreads) void k_nod_bottom(NodBottomArgs<T> A) {
    using Cap = NodBottomCap<T>;
    __shared__ T P0[Cap::nodes], S0[Cap::cells];
    __shared__ __align__(16) T R0[Cap::nodes];          // residual of the first level; the coarsest solve's sums
    __shared__ T P1[Cap::nodes1], S1[Cap::cells1];
    __shared__ __align__(16) T F1[Cap::nodes1], R1[Cap::nodes1];
    __shared__ double rhs2[Cap::coarse], x2[Cap::coarse], mean;
    static_assert(sizeof(R0) >= kMatvecParts * kCoarseMax * sizeof(double), "sums of the coarsest solve");
    static_assert(sizeof(F1) >= kCoarseMax * sizeof(double), "a coarsest level right below the first");
    const NodLevelT<T>&L0 = A.lev[0], &L1 = A.lev[1];
    const bool two = A.nlev > 2;
    const NodLevelT<T>& Lc = A.lev[two ? 2 : 1];
    const int nc = (int)Lc.nodes();
    // the coarsest level's right-hand side and solution: apart below a second level, else in its place
    double* const rhs = two ? rhs2 : reinterpret_cast<double*>(F1);
    double* const x = two ? x2 : reinterpret_cast<double*>(R1);
    T* const Fc = two ? R1 + Cap::nodes1 - Cap::coarse : P1;      // (R1's own values are consumed before)
    NbOwned<T, Cap::own> a;
    NbOwned<T, Cap::own1> o;
    a.load(L0);
    a.load_f(L0, L0.f);
    nb_load_sigma(L0, S0);
    for (int e = threadIdx.x; e < (int)L0.nodes(); e += kNodBottomThreads) P0[e] = T(0);
    if (two) {
        o.load(L1);
        nb_load_sigma(L1, S1);
        for (int e = threadIdx.x; e < (int)L1.nodes(); e += kNodBottomThreads) P1[e] = T(0);
    }
    __syncthreads();
    for (int visit = 0; visit < 2; ++visit) {
        if (visit) nb_prolong(L0, P0, L1, P1);          // two == false: the coarsest solution is in P1 too
        a.sweeps(L0, P0, S0, visit ? A.post : A.pre);
        if (visit) break;
        a.residual(L0, P0, S0, R0);
        nb_restrict(L0, R0, L1, two ? F1 : Fc);
        for (int v1 = 0; v1 < 2; ++v1) {
            if (two && v1) nb_prolong(L1, P1, Lc, Fc);
            if (two) {
                if (!v1) o.load_f(L1, F1);
                o.sweeps(L1, P1, S1, v1 ? A.post : A.pre);
            }
            if (v1) break;
            if (two) {
                o.residual(L1, P1, S1, F1);             // its right-hand side is in registers
                nb_restrict(L1, F1, Lc, Fc);
            }
            for (int c = threadIdx.x; c < nc; c += kNodBottomThreads) rhs[c] = (double)Fc[c];
            __syncthreads();
            dense_solve<kNodBottomThreads>(nc, 1, A.minv, rhs, x, reinterpret_cast<double*>(R0), &mean);
            for (int c = threadIdx.x; c < nc; c += kNodBottomThreads) Fc[c] = (T)x[c];
            __syncthreads();
        }
    }
    for (int e = threadIdx.x; e < (int)L0.nodes(); e += kNodBottomThreads) L0.phi[e] = P0[e];
}

// Grid of a point loop over an X x Y x Z box: at most 2048 workgroups (the
// partial rows), the planes shared out among them.
inline dim3 point_grid(int X, int Y, int Z) {
    const int gx = std::min((X + kPtX - 1) / kPtX, 2048);
    const int gy = std::max(1, std::min((Y + kPtY - 1) / kPtY, 2048 / gx));
    const int gz = std::max(1, std::min(Z, 2048 / (gx * gy)));
    return dim3(gx, gy, gz);
}
inline int grid_blocks(dim3 g) { return (int)(g.x * g.y * g.z); }

inline int nod_partial_blocks(size_t N) {
    size_t b = (N + kNodBlock - 1) / kNodBlock;
    return (int)std::min<size_t>(b, 2048);
}

inline dim3 grid3(int x, int y, int z, dim3 block) {
    return dim3((x + block.x - 1) / block.x, (y + block.y - 1) / block.y, (z + block.z - 1) / block.z);
}

}  // namespace
}  // namespace mg

// ============================================================================
// host side: hierarchy and C ABI
// ============================================================================
using namespace mg;

struct nodal_hierarchy {
    mg_params p{};
    int nlev = 0;
    NodLevel lev[kMaxLevels];
    // mixed precision: FP32 mirrors of every level (sigma, phi, f, phi2),
    // the inner V-cycle's arrays
    bool mixed = false;
    NodLevelT<float> lev32[kMaxLevels];
    void* ws = nullptr;
    double* minv = nullptr;
    double* partials = nullptr;
    double* scal = nullptr;
    double* host = nullptr;
    bool coeffs_valid = false;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    // One V-cycle plus the finest residual norm as a
    // replayable hipGraph on the hierarchy's own stream, keyed by the sweep
    // counts and every level's phi buffers at the start of the cycle (the
    // fused sweeps swap them; with an even number of sweeps a cycle they
    // come back, so one capture serves every cycle of every solve).
    // Off unless asked for: slower than separate launches enqueued ahead (64^3
    // 1128 us a projection against 1074, 128^3 2011 against 1938).
    bool graphs_on = false;
    bool bottom_on = true;      // the coarse levels that fit in LDS run in one workgroup (k_nod_bottom)
    hipStream_t gstream = nullptr;
    hipEvent_t gev = nullptr;
    hipGraphExec_t cycle_exec = nullptr;
    int cycle_pre = -1, cycle_post = -1;
    std::vector<void*> cycle_bufs;
};

namespace {

int nod_count_levels(const mg_params* p) {
    int nx = p->n[0], ny = p->n[1], nz = p->n[2];
    if (nx < 1 || ny < 1 || nz < 1) return 0;
    int n = 1;
    while (nx % 2 == 0 && ny % 2 == 0 && nz % 2 == 0 && (long long)nx * ny * nz > kCoarsenMin && n < kMaxLevels) {
        nx /= 2;
        ny /= 2;
        nz /= 2;
        ++n;
    }
    const long long nodes = (long long)(nx + (p->bc[0] == MG_BC_PERIODIC ? 0 : 1)) *
                            (ny + (p->bc[1] == MG_BC_PERIODIC ? 0 : 1)) * (nz + (p->bc[2] == MG_BC_PERIODIC ? 0 : 1));
    return nodes <= kCoarseMax ? n : 0;
}

// Partial-sum rows: of the point loops, and of the finest level's residual norm.
size_t nod_partial_rows(const NodLevel& L0) {
    return std::max<size_t>(2048, (size_t)nod_resid_grid(L0, L0.Nz, false).blocks());
}

// Level shapes of a hierarchy of nl levels for p (into lev), and the device
// bytes it needs: per level sigma on cells and phi, f, phi2 on nodes (in
// mixed precision also FP32 copies of all four); the coarsest level's dense
// inverse, the partial rows and the scalar block.
size_t nod_layout(const mg_params* p, int nl, NodLevel* lev) {
    size_t bytes = 0;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    for (int l = 0; l < nl; ++l) {
        NodLevel& L = lev[l];
        L.nx = p->n[0] >> l;
        L.ny = p->n[1] >> l;
        L.nz = p->n[2] >> l;
        L.px = p->bc[0] == MG_BC_PERIODIC;
        L.py = p->bc[1] == MG_BC_PERIODIC;
        L.pz = p->bc[2] == MG_BC_PERIODIC;
        L.Nx = L.nx + (L.px ? 0 : 1);
        L.Ny = L.ny + (L.py ? 0 : 1);
        L.Nz = L.nz + (L.pz ? 0 : 1);
        L.h = p->dx * (double)(1 << l);
        bytes += al(L.cells() * 8) + 3 * al(L.nodes() * 8);
        if (p->precision == MG_MIXED) bytes += al(L.cells() * 4) + 3 * al(L.nodes() * 4);
    }
    const size_t nc = lev[nl - 1].nodes();
    bytes += al(nc * nc * 8) + al(nod_partial_rows(lev[0]) * kReduceWidth * 8) + al(64 * 8);
    return bytes;
}

#define NHIP(expr)                                                        \
    do {                                                                  \
        hipError_t e_ = (expr);                                           \
        if (e_ != hipSuccess) return hip_fail(e_, #expr, __LINE__);       \
    } while (0)

// Fused-sweep tiles: 56 x (2 pairs - 8) nodes, tz planes per chunk.
struct NodSweepCfg {
    int pairs, tz;
};
constexpr int kNumNodSweepCfg = 8;
constexpr NodSweepCfg kNodSweepCfgs[kNumNodSweepCfg] = {{8, 2},   {8, 4},   {8, 8},   {8, 16},
                                                       {12, 16}, {12, 32}, {16, 32}, {16, 64}};
std::atomic<int> g_nod_cfg{-1};                  // forced configuration (-1: the rule below)

// Configuration of a level's sweep by its nodes.  Small levels are short of
// workgroups and bound by the steps of one march, so they take few planes per
// chunk; large ones are bound by instruction issue and HBM, where the halo
// (rows and the repeated top plane) is what a bigger tile and longer chunk
// save.  us per sweep in FP64, this choice / the next better one: 32^3 nodes
// 7.0 / 8.9 (8 pairs x 4 planes), 64^3 9.4 / 10.4 (8 x 2), 128^3 26.4 / 28.1
// (12 x 16; with the prolongation, whose 132 registers let 8-pair workgroups
// no longer share a compute unit, 30.6 with 12 x 16 / 41 with 8 x 8), 192^3
// 61 / 66 (8 x 16), 256^3 144 / 149 (16 x 32); in FP32 64^3 7.3, 128^3 18.2,
// 192^3 40, 256^3 65 / 71 (12 x 32), 384 x 384 x 256 163.
template <typename T>
int nod_sweep_config(const NodLevelT<T>& L, bool prolong) {
    const double n = (double)L.nodes();
    if (n < 1e5) return 0;
    if (n < 1e6) return 1;
    if (sizeof(T) == 4) return n < 4e6 ? 2 : 4;
    if (n < 4e6) return prolong ? 4 : 2;
    return n < 12e6 ? 6 : 7;
}

template <typename T>
hipError_t launch_nod_sweep(const NodLevelT<T>& L, T* out, int cfg, const NodLevelT<T>* coarse, hipStream_t st) {
    const NodSweepCfg& c = kNodSweepCfgs[cfg];
    if (c.pairs == 8) return launch_nod_sweep_t<T, 8>(L, out, c.tz, coarse, st);
    if (c.pairs == 12) return launch_nod_sweep_t<T, 12>(L, out, c.tz, coarse, st);
    return launch_nod_sweep_t<T, 16>(L, out, c.tz, coarse, st);
}

// The levels a V-cycle in T runs on: the FP64 hierarchy, or its FP32 mirrors.
template <typename T>
NodLevelT<T>* nod_levels(nodal_hierarchy* H);
template <>
NodLevelT<double>* nod_levels<double>(nodal_hierarchy* H) { return H->lev; }
template <>
NodLevelT<float>* nod_levels<float>(nodal_hierarchy* H) { return H->lev32; }

// First level (>= 1, above the coarsest) that the bottom kernel takes with
// every coarser one, or -1: the first that fits.  One level lower, with the
// march above it, is slower for first levels of 16 x 16 x 17 nodes (32^3 cells
// 0.79 ms for 0.76, 64^3 1.05 for 1.02) and 12 x 12 x 13 (48^3 0.98 for 0.89,
// mixed 0.93 for 0.85), faster only for the largest that FP32 takes (24 x 16 x
// 21, 96x64x80 mixed 1.11 for 1.21).
template <typename T>
int nod_bottom_start(const nodal_hierarchy* H) {
    using Cap = NodBottomCap<T>;
    const NodLevelT<T>* lev = nod_levels<T>(const_cast<nodal_hierarchy*>(H));
    auto fits = [](const NodLevelT<T>& L, int nodes, int cells, int own) {
        const int N[3] = {L.Nx, L.Ny, L.Nz};
        return std::max({L.Nx, L.Ny, L.Nz}) < 1024 && L.nodes() <= (size_t)nodes && nod_bordered(N) <= cells &&
               nod_colour_max(L.Nx, L.Ny, L.Nz) <= own * kNodBottomThreads;
    };
    for (int l = std::max(1, H->nlev - 3); l + 1 < H->nlev; ++l) {
        if (!fits(lev[l], Cap::nodes, Cap::cells, Cap::own)) continue;
        if (H->nlev - l == 3 && (!fits(lev[l + 1], Cap::nodes1, Cap::cells1, Cap::own1) ||
                                 lev[l + 2].nodes() > (size_t)Cap::coarse))
            continue;
        return l;
    }
    return -1;
}

// Whether level l is one of the bottom kernel's: launched one by one (the
// bottom off) these keep the per-node sums that it repeats bit for bit.
template <typename T>
bool nod_in_bottom(const nodal_hierarchy* H, int l) {
    const int b = nod_bottom_start<T>(H);
    return b >= 0 && l >= b;
}

// Whether level l takes the fused out-of-place sweep (its two phi buffers
// swap): wherever the march fits above the bottom kernel's levels.
template <typename T>
bool nod_fused(const nodal_hierarchy* H, int l) {
    return nod_sweep_fits(nod_levels<T>(const_cast<nodal_hierarchy*>(H))[l]) && !nod_in_bottom<T>(H, l);
}

// Sweeps on level l: fused, the first one of phi + P C.phi where coarse is
// given, else one in-place launch per colour.
template <typename T = double>
int nod_smooth(nodal_hierarchy* H, int l, int nsweeps, hipStream_t st, const NodLevelT<T>* coarse = nullptr) {
    NodLevelT<T>& L = nod_levels<T>(H)[l];
    if (nod_fused<T>(H, l)) {
        const int forced = g_nod_cfg.load();
        for (int s = 0; s < nsweeps; ++s) {
            const NodLevelT<T>* c = s == 0 ? coarse : nullptr;
            NHIP(launch_nod_sweep(L, L.phi2, forced >= 0 ? forced : nod_sweep_config(L, c != nullptr), c, st));
            std::swap(L.phi, L.phi2);
        }
        return MG_OK;
    }
    const dim3 block(64, 2, 2);
    const dim3 grid = grid3(L.Nx, (L.Ny + 1) / 2, (L.Nz + 1) / 2, block);
    for (int s = 0; s < nsweeps; ++s)
        for (int col = 0; col < 4; ++col) hipLaunchKernelGGL(k_nod_gs<T>, grid, block, 0, st, L, col);
    NHIP(hipGetLastError());
    return MG_OK;
}

template <typename T = double>
int nod_resid_restrict(nodal_hierarchy* H, int l, hipStream_t st) {
    const NodLevelT<T>& F = nod_levels<T>(H)[l];
    const NodLevelT<T>& C = nod_levels<T>(H)[l + 1];
    if (nod_in_bottom<T>(H, l)) {
        hipLaunchKernelGGL(k_nod_restrict_each<T>, dim3(((int)C.nodes() + 63) / 64), dim3(64), 0, st, F, C);
        NHIP(hipGetLastError());
        return MG_OK;
    }
    NHIP((launch_nod_resid<T, kNodRestrict>(F, C, nullptr, NodRefine{}, nullptr, st)));
    return MG_OK;
}

template <typename T = double>
int nod_prolong(nodal_hierarchy* H, int l, hipStream_t st) {
    const NodLevelT<T>& F = nod_levels<T>(H)[l];
    const NodLevelT<T>& C = nod_levels<T>(H)[l + 1];
    const dim3 block(32, 4, 2);
    hipLaunchKernelGGL(k_nod_prolong<T>, grid3(C.Nx, C.Ny, C.Nz, block), block, 0, st, F, C);
    NHIP(hipGetLastError());
    return MG_OK;
}

hipError_t nod_coarse_solve(int n, const double* minv, const double* f, double* phi, hipStream_t st) {
    return launch_coarse_solve(n, minv, f, phi, st, 1);
}
hipError_t nod_coarse_solve(int n, const double* minv, const float* f, float* phi, hipStream_t st) {
    return launch_coarse_solve_f32(n, minv, f, phi, st, 1);
}

// V-cycle from level l in T (the coarsest solve applies the FP64 inverse).
template <typename T = double>
int nod_vcycle(nodal_hierarchy* H, int l, hipStream_t st) {
    if (H->bottom_on && l > 0 && l == nod_bottom_start<T>(H)) {
        NodBottomArgs<T> a{};
        a.nlev = H->nlev - l;
        for (int b = 0; b < a.nlev; ++b) a.lev[b] = nod_levels<T>(H)[l + b];
        a.minv = H->minv;
        a.pre = H->p.pre_sweeps;
        a.post = H->p.post_sweeps;
        hipLaunchKernelGGL(k_nod_bottom<T>, dim3(1), dim3(kNodBottomThreads), 0, st, a);
        NHIP(hipGetLastError());
        return MG_OK;
    }
    if (l == H->nlev - 1) {
        const NodLevelT<T>& L = nod_levels<T>(H)[l];
        NHIP(nod_coarse_solve((int)L.nodes(), H->minv, L.f, L.phi, st));
        return MG_OK;
    }
    int rc = nod_smooth<T>(H, l, H->p.pre_sweeps, st);
    if (rc) return rc;
    rc = nod_resid_restrict<T>(H, l, st);
    if (rc) return rc;
    rc = nod_vcycle<T>(H, l + 1, st);
    if (rc) return rc;
    if (H->p.post_sweeps > 0 && nod_fused<T>(H, l))
        return nod_smooth<T>(H, l, H->p.post_sweeps, st, &nod_levels<T>(H)[l + 1]);
    rc = nod_prolong<T>(H, l, st);
    if (rc) return rc;
    return nod_smooth<T>(H, l, H->p.post_sweeps, st);
}

// sigma on every level from rho and beta0, coarsest inverse; partial rows
// of the input checks reduced into slot kSlotRhs (bad, #non-finite), enqueued.
int nod_build(nodal_hierarchy* H, const double* rho, const double* b0c, hipStream_t st) {
    const NodLevel& L0 = H->lev[0];
    const dim3 sg = point_grid(L0.nx, L0.ny, L0.nz);
    hipLaunchKernelGGL(k_nod_sigma, sg, dim3(kPtX, kPtY), 0, st, L0, rho, b0c, H->partials);
    NHIP(hipGetLastError());
    NHIP(launch_reduce(H->partials, grid_blocks(sg), H->scal + kSlotRhs * kReduceWidth, st));
    const dim3 block(32, 4, 2);
    for (int l = 0; l + 1 < H->nlev; ++l) {
        const NodLevel& C = H->lev[l + 1];
        hipLaunchKernelGGL(k_nod_avg_sigma, grid3(C.nx, C.ny, C.nz, block), block, 0, st, H->lev[l], C);
    }
    NHIP(launch_nod_coarse_setup(H->lev[H->nlev - 1], H->minv, H->partials, st));
    return MG_OK;
}

// The checks of rho and beta0 in slot kSlotRhs on the host, nonfin more
// non-finite values among the other inputs.
int nod_check(nodal_hierarchy* H, double nonfin) {
    const double* q = H->host + kSlotRhs * kReduceWidth;
    if (q[3] > 0.0 || nonfin > 0.0) {
        set_error("non-finite value in rho, beta0, U or S");
        return MG_ERR_NONFINITE;
    }
    if (q[2] > 0.0) {
        set_error("rho and beta0 must be positive");
        return MG_ERR_INVALID_ARG;
    }
    H->coeffs_valid = true;
    return MG_OK;
}

int nod_read(nodal_hierarchy* H, int slot, int rows, hipStream_t st) {
    NHIP(hipMemcpyAsync(H->host + slot * kReduceWidth, H->scal + slot * kReduceWidth,
                        rows * kReduceWidth * sizeof(double), hipMemcpyDeviceToHost, st));
    NHIP(hipStreamSynchronize(st));
    return MG_OK;
}

int nod_coefficients(nodal_hierarchy* H, const double* rho, const double* b0c, hipStream_t st) {
    int rc = nod_build(H, rho, b0c, st);
    if (!rc) rc = nod_read(H, kSlotRhs, 1, st);
    return rc ? rc : nod_check(H, 0.0);
}

// The iterations of a solve (run_ahead), each of `step` V-cycles, `enqueue`
// putting one on the stream that `stream` then names.
template <typename E, typename Q>
int nod_cycles(nodal_hierarchy* H, double fnorm, mg_stats* S_, bool ahead, int step, int* status, int* cycles,
               double* rel, bool* over, E&& enqueue, Q&& stream) {
    *status = MG_ERR_NOT_CONVERGED;
    auto rows = [&](const double** r) -> int {
        const hipStream_t st = stream();
        *r = H->host + kSlotRing * kReduceWidth;
        return nod_read(H, kSlotRing, kNormRing, st);
    };
    auto record = [&](int c, double r) {
        if (c >= MG_HIST_MAX) return;
        S_->resid_hist[c] = r;
        S_->hist_len = c + 1;
    };
    int rc = run_ahead(fnorm, H->p.rtol, H->p.max_cycles, ahead, std::pow(kFirstGainNodal, step), kReduceWidth, status,
                       cycles, rel, over, [&](int) { return enqueue(); }, rows, record);
    if (rc == MG_OK && *status == MG_ERR_NONFINITE) set_error("non-finite residual during the solve");
    return rc;
}

// Mixed-precision solve (iterative refinement with the multigrid of Sec. 3
// as its inner solver): each iteration runs one FP32 V-cycle from zero on the
// FP64 residual scaled by the power of two nearest 1/rms(r), adds the FP32
// correction divided by that power of two (exact) to the FP64 phi, and
// recomputes r = f - L phi and its norm in FP64; the stop test is the FP64
// solve's.  Returns MG_OK or a launch error; *status is the solve's.
int nod_solve_mixed(nodal_hierarchy* H, double fnorm, mg_stats* S_, int* status_out, int* cycles_out,
                    double* rel_out, bool ahead, bool* over, hipStream_t st) {
    NodLevel& L0 = H->lev[0];
    NodLevelT<float>& M0 = H->lev32[0];
    const size_t NN = L0.nodes();
    for (int l = 0; l < H->nlev; ++l)
        NHIP(launch_coeff_to_f32(H->lev[l].sig, H->lev32[l].sig, H->lev[l].cells(), st));
    const double s0 = residual_scale(fnorm, NN);
    NHIP(launch_scale_to_f32(L0.f, M0.f, NN, s0, st));       // the residual of phi = 0 is f
    double* scales = H->scal + kSlotScale * kReduceWidth;      // {scale of the FP32 residual, scale for the next}
    H->host[kSlotScale * kReduceWidth] = s0;
    H->host[kSlotScale * kReduceWidth + 1] = s0;
    NHIP(hipMemcpyAsync(scales, H->host + kSlotScale * kReduceWidth, 2 * sizeof(double), hipMemcpyHostToDevice, st));
    int nt = 0;
    int status = MG_ERR_NOT_CONVERGED, cycles = 0;
    double rel = 1.0;
    // nodal default one: its FP32 V-cycle costs several refinement passes
    // (256^3: two per step took 8.90 ms against 8.19 with one)
    const int inner = H->p.inner_cycles > 0 ? H->p.inner_cycles : 1;
    auto cycle = [&]() -> int {
        NHIP(launch_fill<float>(M0.phi, NN, 0.0f, st));
        for (int c = 0; c < inner; ++c) {                 // the FP32 correction: V-cycles from zero
            int rc = nod_vcycle<float>(H, 0, st);
            if (rc) return rc;
        }
        // phi += corr / s, r = f - L phi with its norm rows, FP32 r for the
        // next cycle, in one pass (phi out of place); the reduction then
        // advances the scales
        const NodRefine ra{M0.phi, scales, L0.phi2, M0.f};
        NHIP((launch_nod_resid<double, kNodRefine>(L0, L0, H->partials, ra, &nt, st)));
        std::swap(L0.phi, L0.phi2);
        NHIP(launch_reduce_scale(H->partials, nt, H->scal + kSlotRes * kReduceWidth, scales, NN, st,
                                 norm_ring(H->scal)));
        return MG_OK;
    };
    int rc = nod_cycles(H, fnorm, S_, ahead, inner, &status, &cycles, &rel, over, cycle, [&] { return st; });
    if (rc) return rc;
    *status_out = status;
    *cycles_out = cycles;
    *rel_out = rel;
    return MG_OK;
}

// FP64 solve: V-cycles on phi, each with the finest residual norm after it,
// from a captured graph where the levels' buffers come back.
int nod_solve(nodal_hierarchy* H, double fnorm, mg_stats* S_, int* status, int* cycles, double* rel, bool ahead,
              bool* over, hipStream_t st) {
    NodLevel& L0 = H->lev[0];
    bool on_graph = false;
    auto cycle = [&](hipStream_t s) -> int {
        int r2 = nod_vcycle(H, 0, s);
        if (r2) return r2;
        int nt = 0;
        NHIP((launch_nod_resid<double, kNodNorm>(L0, L0, H->partials, NodRefine{}, &nt, s)));
        NHIP(launch_reduce(H->partials, nt, H->scal + kSlotRes * kReduceWidth, s, norm_ring(H->scal)));
        return MG_OK;
    };
    // a captured cycle bakes in the levels' phi buffers: replayable when
    // every level's buffers come back (an even number of sweeps a cycle)
    const bool graphs = H->graphs_on && (H->p.pre_sweeps + H->p.post_sweeps) % 2 == 0;
    auto enqueue = [&]() -> int {
        if (!graphs) return cycle(st);
        if (!H->gstream) {
            NHIP(hipStreamCreateWithFlags(&H->gstream, hipStreamNonBlocking));
            NHIP(hipEventCreateWithFlags(&H->gev, hipEventDisableTiming));
        }
        if (!on_graph) {                    // after the caller's earlier work
            NHIP(hipEventRecord(H->gev, st));
            NHIP(hipStreamWaitEvent(H->gstream, H->gev, 0));
            on_graph = true;
        }
        std::vector<void*> bufs;
        for (int l = 0; l < H->nlev; ++l) {
            bufs.push_back(H->lev[l].phi);
            bufs.push_back(H->lev[l].phi2);
        }
        bufs.push_back((void*)(intptr_t)g_nod_cfg.load());      // the tiles the capture baked in
        if (!H->cycle_exec || H->cycle_pre != H->p.pre_sweeps || H->cycle_post != H->p.post_sweeps ||
            H->cycle_bufs != bufs) {
            if (H->cycle_exec) {
                NHIP(hipStreamSynchronize(H->gstream));      // a cycle enqueued ahead may still run it
                hipGraphExecDestroy(H->cycle_exec);
                H->cycle_exec = nullptr;
            }
            NHIP(hipStreamBeginCapture(H->gstream, hipStreamCaptureModeRelaxed));
            int r2 = cycle(H->gstream);
            hipGraph_t g = nullptr;
            hipError_t e = hipStreamEndCapture(H->gstream, &g);
            if (r2) {
                if (g) hipGraphDestroy(g);
                return r2;
            }
            if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture", __LINE__);
            e = hipGraphInstantiate(&H->cycle_exec, g, nullptr, nullptr, 0);
            hipGraphDestroy(g);
            if (e != hipSuccess) {
                H->cycle_exec = nullptr;
                return hip_fail(e, "hipGraphInstantiate", __LINE__);
            }
            H->cycle_pre = H->p.pre_sweeps;
            H->cycle_post = H->p.post_sweeps;
            H->cycle_bufs = bufs;
        }
        NHIP(hipGraphLaunch(H->cycle_exec, H->gstream));
        return MG_OK;
    };
    return nod_cycles(H, fnorm, S_, ahead, 1, status, cycles, rel, over, enqueue,
                      [&] { return on_graph ? H->gstream : st; });
}

int nod_project(nodal_hierarchy* H, const double* rho, const double* b0c, const double* S, double* u, double* v,
                double* w, double* phi_out, mg_stats* S_, hipStream_t st) {
    std::memset(S_, 0, sizeof *S_);
    S_->nlevels = H->nlev;
    NHIP(hipEventRecord(H->ev0, st));
    int rc = nod_build(H, rho, b0c, st);
    if (rc) return S_->status = rc;
    NodLevel& L0 = H->lev[0];
    const size_t NN = L0.nodes();
    // f, then its mean removed and its norm, and one look at all the rows
    NodResidGrid g = nod_resid_grid(L0, L0.Nz, false);
    g.ntx = (L0.Nx + kRhsTX - 1) / kRhsTX;        // no more rows than the residual's
    hipLaunchKernelGGL(k_nod_rhs, dim3(g.blocks()), dim3(64, kNodResidWaves), 0, st, L0, b0c, u, v, w, S, g.tz, g.ntx,
                       g.nty, H->partials);
    NHIP(hipGetLastError());
    NHIP(launch_reduce(H->partials, g.blocks(), H->scal + kSlotNorm * kReduceWidth, st));
    int np = 0;
    NHIP(launch_shift_norm(Shape{L0.Nx, L0.Ny, L0.Nz}, L0.f, 0.0, H->partials, &np, st,
                           H->scal + kSlotNorm * kReduceWidth));
    NHIP(launch_reduce(H->partials, np, H->scal + kSlotRes * kReduceWidth, st));
    static_assert(kSlotNorm == kSlotRhs + 1 && kSlotRes == kSlotRhs + 2, "read together");
    rc = nod_read(H, kSlotRhs, 3, st);
    if (rc) return S_->status = rc;
    const double* q = H->host + kSlotNorm * kReduceWidth;
    rc = nod_check(H, q[3]);
    if (rc) return S_->status = rc;
    const double sf = q[0], saf = q[1];
    S_->sum_f = sf;
    S_->sum_abs_f = saf;
    if (!std::isfinite(sf) || !std::isfinite(saf)) {
        set_error("non-finite right-hand side");
        return S_->status = MG_ERR_NONFINITE;
    }
    if (std::fabs(sf) > 1e-8 * saf) {
        set_error("incompatible right-hand side: |sum f| > 1e-8 sum |f|");
        return S_->status = MG_ERR_INCOMPATIBLE_RHS;
    }
    S_->mean_removed = sf / (double)NN;
    const double fnorm = std::sqrt(H->host[kSlotRes * kReduceWidth]);
    S_->norm_f = fnorm;
    int status = MG_OK, cycles = 0;
    double rel = 0.0;
    // the cycles' wall time, their last look at the norms included, is the
    // device time of the cycles
    const auto t_s0 = std::chrono::steady_clock::now();
    // looking ahead first; again without where that went beyond convergence
    for (int pass = 0; pass < 2; ++pass) {
        bool over = false;
        cycles = 0;
        rel = 0.0;
        NHIP(launch_fill<double>(L0.phi, NN, 0.0, st));
        NHIP(launch_reduce(H->partials, 0, H->scal + kSlotRes * kReduceWidth, st, norm_ring(H->scal), true));
        S_->resid_hist[0] = fnorm > 0.0 ? 1.0 : 0.0;
        S_->rel_resid0 = S_->resid_hist[0];
        S_->hist_len = 1;
        if (fnorm > 0.0 && H->p.rtol < 1.0) {
            rel = 1.0;
            rc = H->mixed ? nod_solve_mixed(H, fnorm, S_, &status, &cycles, &rel, pass == 0, &over, st)
                          : nod_solve(H, fnorm, S_, &status, &cycles, &rel, pass == 0, &over, st);
            if (rc) return S_->status = rc;
            if (!H->mixed && cycles == 0) rel = 0.0;
        }
        if (!over) break;
    }
    if (H->gstream) {                       // the caller's stream continues after the graph work
        NHIP(hipEventRecord(H->gev, H->gstream));
        NHIP(hipStreamWaitEvent(st, H->gev, 0));
    }
    S_->ms_smooth = cycles > 0 ? std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t_s0).count()
                               : 0.0;
    S_->cycles = cycles;
    S_->rel_resid = rel;
    if (status != MG_OK && status != MG_ERR_NOT_CONVERGED) return S_->status = status;
    NHIP(launch_sum(Shape{L0.Nx, L0.Ny, L0.Nz}, L0.phi, H->partials, &np, st));
    NHIP(launch_reduce(H->partials, np, H->scal + kSlotPhi * kReduceWidth, st));
    const double* psum = H->scal + kSlotPhi * kReduceWidth;
    const dim3 block(32, 4, 2);
    hipLaunchKernelGGL(k_nod_correct, grid3(L0.nx, L0.ny, L0.nz, block), block, 0, st, L0, rho, psum, u, v, w);
    if (phi_out)
        hipLaunchKernelGGL(k_nod_shift_out, dim3(nod_partial_blocks(NN)), dim3(kNodBlock), 0, st, NN, L0.phi, psum,
                           phi_out);
    NHIP(hipGetLastError());
    NHIP(hipEventRecord(H->ev1, st));
    NHIP(hipMemcpyAsync(H->host + kSlotPhi * kReduceWidth, psum, sizeof(double), hipMemcpyDeviceToHost, st));
    NHIP(hipStreamSynchronize(st));
    S_->phi_mean = H->host[kSlotPhi * kReduceWidth] / (double)NN;
    float ms = 0.f;
    hipEventElapsedTime(&ms, H->ev0, H->ev1);
    S_->ms_total = ms;
    S_->ms_other = std::max(0.0, S_->ms_total - S_->ms_smooth);
    S_->status = status;
    if (status == MG_ERR_NOT_CONVERGED) set_error("maximum number of cycles reached");
    return status;
}

}  // namespace

namespace mg {

size_t nodal_bytes(const mg_params* p) {
    if (!p || validate_params(p) != MG_OK) return 0;
    for (int d = 0; d < 3; ++d)
        if (p->bc[d] != MG_BC_PERIODIC && p->bc[d] != MG_BC_WALL) return 0;
    const int nl = nod_count_levels(p);
    if (nl == 0) return 0;
    NodLevel lev[kMaxLevels];
    return nod_layout(p, nl, lev);
}

void nodal_rebind(nodal_handle h, const mg_params* p) { h->p = *p; }

}  // namespace mg

extern "C" {

int nodal_tune_sweep(int32_t cfg) {
    if (cfg < -1 || cfg >= kNumNodSweepCfg) {
        set_error("nodal sweep configuration out of range");
        return MG_ERR_INVALID_ARG;
    }
    g_nod_cfg.store(cfg);
    return MG_OK;
}

int32_t nodal_num_levels_for(const mg_params* p) {
    if (!p) return 0;
    for (int d = 0; d < 3; ++d)
        if (p->bc[d] != MG_BC_PERIODIC && p->bc[d] != MG_BC_WALL) return 0;
    return nod_count_levels(p);
}

int nodal_setup(const mg_params* p, nodal_handle* out) {
    if (!out || !p) {
        set_error("null argument to nodal_setup");
        return MG_ERR_INVALID_ARG;
    }
    *out = nullptr;
    int st = validate_params(p);
    if (st != MG_OK) return st;
    for (int d = 0; d < 3; ++d)
        if (p->bc[d] != MG_BC_PERIODIC && p->bc[d] != MG_BC_WALL) {
            set_error("the nodal projection takes periodic or wall boundaries");
            return MG_ERR_INVALID_ARG;
        }
    if (p->precision != MG_FP64 && p->precision != MG_MIXED) {
        set_error("unknown precision");
        return MG_ERR_INVALID_ARG;
    }
    const int nl = nod_count_levels(p);
    if (nl == 0) {
        set_error("shape not solvable: the coarsest nodal level would exceed 512 nodes");
        return MG_ERR_BAD_SIZE;
    }
    nodal_hierarchy* H = new (std::nothrow) nodal_hierarchy();
    if (!H) return MG_ERR_OOM;
    H->p = *p;
    H->nlev = nl;
    const size_t bytes = nod_layout(p, nl, H->lev);
    if (hipMalloc(&H->ws, bytes) != hipSuccess) {
        (void)hipGetLastError();
        delete H;
        set_error("hipMalloc of the nodal hierarchy failed");
        return MG_ERR_OOM;
    }
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t nc = H->lev[nl - 1].nodes();
    const size_t prow = nod_partial_rows(H->lev[0]);
    char* b = (char*)H->ws;
    auto take = [&](size_t n) {
        char* q = b;
        b += al(n);
        return (double*)q;
    };
    for (int l = 0; l < nl; ++l) {
        NodLevel& L = H->lev[l];
        L.sig = take(L.cells() * 8);
        L.phi = take(L.nodes() * 8);
        L.f = take(L.nodes() * 8);
        L.phi2 = take(L.nodes() * 8);
    }
    H->mixed = p->precision == MG_MIXED;
    if (H->mixed) {
        auto take32 = [&](size_t n) { return reinterpret_cast<float*>(take(n * 4)); };
        for (int l = 0; l < nl; ++l) {
            const NodLevel& L = H->lev[l];
            NodLevelT<float>& M = H->lev32[l];
            M.nx = L.nx; M.ny = L.ny; M.nz = L.nz;
            M.Nx = L.Nx; M.Ny = L.Ny; M.Nz = L.Nz;
            M.px = L.px; M.py = L.py; M.pz = L.pz;
            M.h = L.h;
            M.sig = take32(L.cells());
            M.phi = take32(L.nodes());
            M.f = take32(L.nodes());
            M.phi2 = take32(L.nodes());
        }
    }
    H->minv = take(nc * nc * 8);
    H->partials = take(prow * kReduceWidth * 8);
    H->scal = take(64 * 8);
    if (hipHostMalloc((void**)&H->host, 64 * sizeof(double), hipHostMallocDefault) != hipSuccess) {
        hipFree(H->ws);
        delete H;
        set_error("hipHostMalloc failed");
        return MG_ERR_HIP;
    }
    hipEventCreate(&H->ev0);
    hipEventCreate(&H->ev1);
    *out = H;
    return MG_OK;
}

int nodal_destroy(nodal_handle h) {
    if (!h) return MG_OK;
    if (h->cycle_exec) hipGraphExecDestroy(h->cycle_exec);
    if (h->gstream) hipStreamDestroy(h->gstream);
    if (h->gev) hipEventDestroy(h->gev);
    if (h->ws) hipFree(h->ws);
    if (h->host) hipHostFree(h->host);
    hipEventDestroy(h->ev0);
    hipEventDestroy(h->ev1);
    delete h;
    return MG_OK;
}

int nodal_project(nodal_handle h, const double* rho, const double* beta0_cc, const double* S, double* uc,
                  double* vc, double* wc, double* phi, mg_stats* stats, void* stream) {
    if (!h || !rho || !beta0_cc || !S || !uc || !vc || !wc) {
        set_error("null argument to nodal_project");
        return MG_ERR_INVALID_ARG;
    }
    mg_stats local;
    try {
        return nod_project(h, rho, beta0_cc, S, uc, vc, wc, phi, stats ? stats : &local, (hipStream_t)stream);
    } catch (...) {
        set_error("internal error in nodal_project");
        return MG_ERR_HIP;
    }
}

int nodal_set_coefficients(nodal_handle h, const double* rho, const double* beta0_cc, void* stream) {
    if (!h || !rho || !beta0_cc) {
        set_error("null argument to nodal_set_coefficients");
        return MG_ERR_INVALID_ARG;
    }
    return nod_coefficients(h, rho, beta0_cc, (hipStream_t)stream);
}

int nodal_set_graphs(nodal_handle h, int32_t enable) {
    if (!h) {
        set_error("null handle");
        return MG_ERR_INVALID_ARG;
    }
    h->graphs_on = enable != 0;
    return MG_OK;
}

int nodal_set_bottom(nodal_handle h, int32_t enable) {
    if (!h) {
        set_error("null handle");
        return MG_ERR_INVALID_ARG;
    }
    h->bottom_on = enable != 0;
    if (h->cycle_exec) {                 // a captured cycle baked in the other choice
        hipGraphExecDestroy(h->cycle_exec);
        h->cycle_exec = nullptr;
    }
    return MG_OK;
}

int nodal_level_info(nodal_handle h, int32_t level, int32_t dims[6], double* dx) {
    if (!h || level < 0 || level >= h->nlev || !dims) {
        set_error("bad nodal_level_info arguments");
        return MG_ERR_INVALID_ARG;
    }
    const NodLevel& L = h->lev[level];
    dims[0] = L.Nx;
    dims[1] = L.Ny;
    dims[2] = L.Nz;
    dims[3] = L.nx;
    dims[4] = L.ny;
    dims[5] = L.nz;
    if (dx) *dx = L.h;
    return MG_OK;
}

int nodal_level_copy(nodal_handle h, int32_t level, int32_t array, void* buffer, int32_t to_hierarchy,
                     void* stream) {
    if (!h || level < 0 || level >= h->nlev || !buffer) {
        set_error("bad nodal_level_copy arguments");
        return MG_ERR_INVALID_ARG;
    }
    const NodLevel& L = h->lev[level];
    double* a;
    size_t n;
    switch (array) {
        case MG_NOD_PHI: a = L.phi; n = L.nodes(); break;
        case MG_NOD_F: a = L.f; n = L.nodes(); break;
        case MG_NOD_SIGMA: a = L.sig; n = L.cells(); break;
        default: set_error("bad nodal array id"); return MG_ERR_INVALID_ARG;
    }
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = to_hierarchy ? launch_copy(a, (const double*)buffer, n, st)
                                : launch_copy((double*)buffer, a, n, st);
    if (e != hipSuccess) return hip_fail(e, "nodal_level_copy", __LINE__);
    return MG_OK;
}

int nodal_level_step(nodal_handle h, int32_t level, int32_t step, int32_t arg, void* stream) {
    if (!h || level < 0 || level >= h->nlev) {
        set_error("bad level");
        return MG_ERR_INVALID_ARG;
    }
    if (!h->coeffs_valid) {
        set_error("nodal_level_step before nodal_set_coefficients / nodal_project");
        return MG_ERR_INVALID_ARG;
    }
    hipStream_t st = (hipStream_t)stream;
    const bool has_coarse = level + 1 < h->nlev;
    switch (step) {
        case MG_STEP_SMOOTH: return nod_smooth(h, level, arg, st);
        case MG_STEP_RESID_RESTRICT:
            if (!has_coarse) break;
            return nod_resid_restrict(h, level, st);
        case MG_STEP_PROLONG:
            if (!has_coarse) break;
            return nod_prolong(h, level, st);
        case MG_STEP_COARSE: {
            if (has_coarse) break;
            const NodLevel& L = h->lev[level];
            NHIP(launch_nod_coarse_setup(L, h->minv, h->partials, st));
            NHIP(launch_coarse_solve((int)L.nodes(), h->minv, L.f, L.phi, st, 1));
            return MG_OK;
        }
        default: break;
    }
    set_error("step not available on this level");
    return MG_ERR_INVALID_ARG;
}

}  // extern "C"
