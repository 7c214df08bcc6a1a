// Finest- and coarse-level operations on small levels (gfx950): one workgroup
// per 16 x 8 x 4 cells, no march through planes.
//
// The marching sweep (sweep.hip) pays about 0.65 us per plane step, most of it
// latency, which a level that leaves most CUs idle cannot hide: 6 steps for
// 4 planes.  Here every thread issues all the loads of its red cells (the
// tile and one cell around it, 2.1 times the tile's own red cells) and of its
// black cell at once, straight from global memory, updates the red cells into
// LDS, and after one barrier the black ones: one memory round trip and one
// barrier a sweep, whatever the level's size.  What it gives up is memory
// traffic (each value is fetched by several threads and neighbouring tiles,
// from the caches), so large levels keep the march.  MI355X, sweep / residual +
// restriction: 32^3 FP64 from rho 10.5 -> 6.1 / 9.2 -> 5.0 us (8-plane march
// before), stored 6.1 -> 4.7 / 6.0 -> 5.2 us (4-plane march, one thread per
// coarse cell); a launch that does nothing takes about 2.
//
// The per-cell expressions are the marching sweep's, so a level's values do
// not depend on which of the two runs (only the per-tile norm rows are
// ordered by tile).
#include <hip/hip_runtime.h>

#include "devmath.h"
#include "mg_internal.h"
#include "sweep.h"

namespace mg {
namespace {

constexpr int kTX = kSweepCfgs[kTileCfg].tx, kTY = kSweepCfgs[kTileCfg].ty, kTZ = kSweepCfgs[kTileCfg].tz;
constexpr int kTileThreads = 256;
constexpr int kWX = kTX + 2, kWY = kTY + 2, kWZ = kTZ + 2;       // the tile and one cell around it
constexpr int kRed = kWX / 2 * kWY * kWZ;                        // red cells of that window
constexpr int kRedPer = (kRed + kTileThreads - 1) / kTileThreads;
static_assert(kTX * kTY * kTZ == 2 * kTileThreads, "one black cell and one pair per thread");

// A cell and its neighbours (periodic wrap; beyond a wall the wrapped
// neighbour meets a zero coefficient).  Sides are even, at least 2.
struct Cell {
    int i, j, k;
    unsigned c, xm, xp, ym, yp, zm, zp;      // flat indices (a tiled level is far below 2^32 cells)
};

template <typename T>
__device__ __forceinline__ Cell cell(const SweepArgs<T>& a, int gx, int gy, int gz) {
    auto wrap = [](int g, int n) { return g < 0 ? g + n : (g >= n ? g - n : g); };
    Cell q;
    q.i = wrap(gx, a.nx);
    q.j = wrap(gy, a.ny);
    q.k = wrap(gz, a.nz);
    const unsigned nx = a.nx, plane = nx * a.ny;
    const unsigned row = q.k * plane + q.j * nx;
    q.c = row + q.i;
    q.xm = row + (q.i > 0 ? q.i - 1 : a.nx - 1);
    q.xp = row + (q.i < a.nx - 1 ? q.i + 1 : 0);
    q.ym = q.j > 0 ? q.c - nx : q.c + (a.ny - 1) * nx;
    q.yp = q.j < a.ny - 1 ? q.c + nx : q.c - (a.ny - 1) * nx;
    q.zm = q.k > 0 ? q.c - plane : q.c + (a.nz - 1) * plane;
    q.zp = q.k < a.nz - 1 ? q.c + plane : q.c - (a.nz - 1) * plane;
    return q;
}

// The six face coefficients as loaded: the stored ones, or rho of the cell
// and its neighbours and the beta0 values, from which they follow.
template <typename T, bool kRho>
struct Coeffs {
    T v[kRho ? 7 : 6];
    double b0[kRho ? 3 : 1];
    bool wall[kRho ? 6 : 1];
    __device__ __forceinline__ void load(const SweepArgs<T>& a, const Cell& q) {
        if constexpr (kRho) {
            const unsigned at[7] = {q.xm, q.xp, q.ym, q.yp, q.zm, q.zp, q.c};
#pragma unroll
            for (int d = 0; d < 7; ++d) v[d] = a.rho[at[d]];
            b0[0] = a.b0c[q.k];
            b0[1] = a.b0e[q.k];
            b0[2] = a.b0e[q.k < a.nz - 1 ? q.k + 1 : 0];
            wall[0] = q.i == 0 && !a.px;
            wall[1] = q.i == a.nx - 1 && !a.px;
            wall[2] = q.j == 0 && !a.py;
            wall[3] = q.j == a.ny - 1 && !a.py;
            wall[4] = q.k == 0 && !a.pz;
            wall[5] = q.k == a.nz - 1 && !a.pz;
        } else {
            v[0] = a.bx[q.c];
            v[1] = a.bx[q.xp];
            v[2] = a.by[q.c];
            v[3] = a.by[q.yp];
            v[4] = a.bz[q.c];
            v[5] = a.bz[q.zp];
        }
    }
    __device__ __forceinline__ void get(T (&b)[6]) const {
        if constexpr (kRho) {
#pragma unroll
            for (int d = 0; d < 6; ++d) {
                const T s = d & 1 ? v[6] + v[d] : v[d] + v[6];         // low cell + high cell
                b[d] = wall[d] ? T(0) : pdiv((T)b0[d < 4 ? 0 : d - 3], T(0.5) * s);
            }
        } else {
#pragma unroll
            for (int d = 0; d < 6; ++d) b[d] = v[d];
        }
    }
};

// phi_in around a cell, as the operation reads it: stored, plus the parent's
// coarse value (kInProlong) or plus the scaled FP32 correction (kInCorrect).
template <typename T, int kIn, int N>
struct Around {
    T v[N], e[kIn == kInProlong || kIn == kInCorrect ? N : 1];
    __device__ __forceinline__ void load(const SweepArgs<T>& a, const Cell& q) {
        if (kIn == kInZero) return;
        const unsigned at[7] = {q.xm, q.xp, q.ym, q.yp, q.zm, q.zp, q.c};
#pragma unroll
        for (int d = 0; d < N; ++d) v[d] = a.phi_in[at[d]];
        if constexpr (kIn == kInProlong) {
            const unsigned hx = a.nx >> 1, hp = hx * (a.ny >> 1);
            const int im = q.i > 0 ? q.i - 1 : a.nx - 1, ip = q.i < a.nx - 1 ? q.i + 1 : 0;
            const int jm = q.j > 0 ? q.j - 1 : a.ny - 1, jp = q.j < a.ny - 1 ? q.j + 1 : 0;
            const int km = q.k > 0 ? q.k - 1 : a.nz - 1, kp = q.k < a.nz - 1 ? q.k + 1 : 0;
            const int X[7] = {im, ip, q.i, q.i, q.i, q.i, q.i}, Y[7] = {q.j, q.j, jm, jp, q.j, q.j, q.j};
            const int Z[7] = {q.k, q.k, q.k, q.k, km, kp, q.k};
#pragma unroll
            for (int d = 0; d < N; ++d) e[d] = a.phic[(Z[d] >> 1) * hp + (Y[d] >> 1) * hx + (X[d] >> 1)];
        }
        if constexpr (kIn == kInCorrect) {
#pragma unroll
            for (int d = 0; d < N; ++d) e[d] = (T)a.corr[at[d]];
        }
    }
    __device__ __forceinline__ void get(T (&p)[N], T cscale) const {
#pragma unroll
        for (int d = 0; d < N; ++d) {
            if (kIn == kInZero) p[d] = T(0);
            else if (kIn == kInPlain) p[d] = v[d];
            else if (kIn == kInProlong) p[d] = v[d] + e[d];
            else p[d] = v[d] + cscale * e[d];
        }
    }
};

template <typename T>
__device__ __forceinline__ T face_sum(const T (&b)[6]) {
    T d = b[0] + b[1];
    d = d + b[2];
    d = d + b[3];
    d = d + b[4];
    return d + b[5];
}

template <typename T>
__device__ __forceinline__ T weighted_sum(const T (&b)[6], const T* p) {
    T num = b[0] * p[0];
    num = num + b[1] * p[1];
    num = num + b[2] * p[2];
    num = num + b[3] * p[3];
    num = num + b[4] * p[4];
    return num + b[5] * p[5];
}

// p: the six neighbours and the cell itself; g: its boundary diagonal (kBnd)
template <typename T, bool kBnd>
__device__ __forceinline__ T residual(const T (&b)[6], const T (&p)[7], T f, T g, T ih2) {
    T r = b[0] * (p[0] - p[6]);
#pragma unroll
    for (int d = 1; d < 6; ++d) r = r + b[d] * (p[d] - p[6]);
    if (kBnd) r = r - g * p[6];
    return f - r * ih2;
}

// FP32: the fused sweep's division on the levels that the marching sweep
// takes too, else that of the per-colour kernels and the bottom.
template <typename T>
__device__ __forceinline__ T divide(T x, T y, int march_div) {
    if (sizeof(T) == 8) return qdiv(x, y);
    return march_div ? pdiv(x, y) : qdiv(x, y);
}

// Sum of v over the workgroup in a fixed order, to row[0] (the others 0).
__device__ __forceinline__ void norm_row(double v, double* red, double* row) {
    for (int w = 32; w > 0; w >>= 1) v += __shfl_xor(v, w, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        row[0] = (red[0] + red[1]) + (red[2] + red[3]);
        row[1] = 0.0;
        row[2] = 0.0;
        row[3] = 0.0;
    }
}

template <typename T, bool kRho, int kIn, int kOp, bool kBnd>
__device__ __forceinline__ void tile_sweep(const SweepArgs<T>& a, int tile) {
    constexpr bool kNorm = kOp == kOpSweepNorm;
    __shared__ T sR[kWZ][kWY][kWX];
    __shared__ double red[4];
    const int x0 = (tile % a.ntx) * kTX, y0 = (tile / a.ntx % a.nty) * kTY, z0 = tile / (a.ntx * a.nty) * kTZ;
    const T h2 = a.h2, ih2 = T(1) / a.h2;
    const int t = threadIdx.x;
    // the loads of the red cells and of the black cell, all in flight together
    Cell rq[kRedPer];
    Coeffs<T, kRho> rc[kRedPer];
    Around<T, kIn, 6> rp[kRedPer];
    T rf[kRedPer], rg[kRedPer], rpin[kRedPer];
    int rw[kRedPer];                 // window position, or -1
    bool own[kRedPer];               // a cell of the tile (and of the level)
#pragma unroll
    for (int m = 0; m < kRedPer; ++m) {
        const int e = min(t + m * kTileThreads, kRed - 1);
        const int xi = e % (kWX / 2), r = e / (kWX / 2), wy = r % kWY, wz = r / kWY;
        const int gy = y0 - 1 + wy, gz = z0 - 1 + wz;
        const int wx = 2 * xi + ((x0 - 1 + gy + gz) & 1), gx = x0 - 1 + wx;
        // cells more than one beyond the level (a ragged tile) are not needed
        const bool in = t + m * kTileThreads < kRed && gx <= a.nx && gy <= a.ny && gz <= a.nz;
        own[m] = in && wx >= 1 && wx <= kTX && wy >= 1 && wy <= kTY && wz >= 1 && wz <= kTZ && gx < a.nx &&
                 gy < a.ny && gz < a.nz;
        rw[m] = in ? (wz * kWY + wy) * kWX + wx : -1;
        rq[m] = cell(a, min(gx, a.nx), min(gy, a.ny), min(gz, a.nz));
        rc[m].load(a, rq[m]);
        rp[m].load(a, rq[m]);
        rf[m] = a.f[rq[m].c];
        if (kBnd) rg[m] = a.dg[rq[m].c];
        if (kNorm) rpin[m] = a.phi_in[rq[m].c];
    }
    const int by = t / (kTX / 2) % kTY, bz = t / (kTX / 2 * kTY);
    const int gy = y0 + by, gz = z0 + bz, bx = 2 * (t % (kTX / 2)) + ((x0 + gy + gz + 1) & 1), gx = x0 + bx;
    const bool bin = gx < a.nx && gy < a.ny && gz < a.nz;
    const Cell bq = cell(a, min(gx, a.nx), min(gy, a.ny), min(gz, a.nz));
    Coeffs<T, kRho> bc;
    Around<T, kIn, 7> bp;
    bc.load(a, bq);
    if (kNorm) bp.load(a, bq);
    const T bf = a.f[bq.c];
    const T bg = kBnd ? a.dg[bq.c] : T(0);
    double nrm2 = 0.0;
#pragma unroll
    for (int m = 0; m < kRedPer; ++m) {
        T b[6], p[6];
        rc[m].get(b);
        rp[m].get(p, T(0));
        T den = face_sum(b);
        if (kBnd) den = den + rg[m];
        const T v = divide(weighted_sum(b, p) - h2 * rf[m], den, a.march_div);
        if (rw[m] >= 0) (&sR[0][0][0])[rw[m]] = v;
        if (own[m]) {
            a.phi_out[rq[m].c] = v;
            if (kNorm) {
                const double r = (double)(den * (rpin[m] - v) * ih2);
                nrm2 += r * r;
            }
        }
    }
    T b[6];
    bc.get(b);
    T den = face_sum(b);
    if (kBnd) den = den + bg;
    if (kNorm && bin) {
        T p[7];
        bp.get(p, T(0));
        const double r = (double)residual<T, kBnd>(b, p, bf, bg, ih2);
        nrm2 += r * r;
    }
    __syncthreads();
    const int wx = bx + 1, wy = by + 1, wz = bz + 1;
    const T p[6] = {sR[wz][wy][wx - 1], sR[wz][wy][wx + 1], sR[wz][wy - 1][wx],
                    sR[wz][wy + 1][wx], sR[wz - 1][wy][wx], sR[wz + 1][wy][wx]};
    if (bin) a.phi_out[bq.c] = divide(weighted_sum(b, p) - h2 * bf, den, a.march_div);
    if (kNorm) norm_row(nrm2, red, a.partials + (size_t)tile * kReduceWidth);
}

// Residual of the tile's cells, an x pair per thread: restricted (kOpResidRestrict),
// or of phi_in + corr / scales[0] with the corrected phi, the scaled FP32
// residual and the norm row written (kOpRefine).
template <typename T, bool kRho, int kIn, int kOp, bool kBnd>
__device__ __forceinline__ void tile_residual(const SweepArgs<T>& a, int tile) {
    __shared__ T sr[kTZ][kTY][kTX];
    __shared__ double red[4];
    const int x0 = (tile % a.ntx) * kTX, y0 = (tile / a.ntx % a.nty) * kTY, z0 = tile / (a.ntx * a.nty) * kTZ;
    const T ih2 = T(1) / a.h2;
    const T cscale = kIn == kInCorrect ? (T)(1.0 / a.scales[0]) : T(0);
    const double rscale = kOp == kOpRefine ? a.scales[1] : 0.0;
    const int t = threadIdx.x;
    const int bx = 2 * (t % (kTX / 2)), by = t / (kTX / 2) % kTY, bz = t / (kTX / 2 * kTY);
    const int gx = x0 + bx, gy = y0 + by, gz = z0 + bz;
    const bool in = gx < a.nx && gy < a.ny && gz < a.nz;      // sides are even: a pair is in or out
    Cell q[2];
    Coeffs<T, kRho> co[2];
    Around<T, kIn, 7> ar[2];
    T f[2], g[2] = {T(0), T(0)};
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        q[d] = cell(a, min(gx + d, a.nx), min(gy, a.ny), min(gz, a.nz));
        co[d].load(a, q[d]);
        ar[d].load(a, q[d]);
        f[d] = a.f[q[d].c];
        if (kBnd) g[d] = a.dg[q[d].c];
    }
    double nrm2 = 0.0;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        T b[6], p[7];
        co[d].get(b);
        ar[d].get(p, cscale);
        const T r = residual<T, kBnd>(b, p, f[d], g[d], ih2);
        if (kOp == kOpResidRestrict) sr[bz][by][bx + d] = r;
        if (kOp == kOpRefine && in) {
            const double rd = (double)r;
            nrm2 += rd * rd;
            a.phi_out[q[d].c] = p[6];
            a.r32[q[d].c] = (float)(rscale * rd);
        }
    }
    if (kOp == kOpRefine) norm_row(nrm2, red, a.partials + (size_t)tile * kReduceWidth);
    if (kOp == kOpResidRestrict) {
        __syncthreads();
        if (t >= kTX * kTY * kTZ / 8) return;
        const int I = t % (kTX / 2), J = t / (kTX / 2) % (kTY / 2), K = t / (kTX / 2 * (kTY / 2));
        if (x0 + 2 * I >= a.nx || y0 + 2 * J >= a.ny || z0 + 2 * K >= a.nz) return;
        T s = T(0);
#pragma unroll
        for (int e = 0; e < 8; ++e) s = s + sr[2 * K + (e >> 2)][2 * J + ((e >> 1) & 1)][2 * I + (e & 1)];
        const int hx = a.nx >> 1;
        const size_t C = ((size_t)(z0 / 2 + K) * (a.ny >> 1) + y0 / 2 + J) * hx + x0 / 2 + I;
        a.fc[C] = T(0.125) * s;
        a.phic_out[C] = T(0);
    }
}

template <typename T, bool kRho, int kIn, int kOp, bool kBnd>
__device__ __forceinline__ void tile_body(const SweepArgs<T>& a, int tile) {
    if constexpr (kOp == kOpSweep || kOp == kOpSweepNorm) tile_sweep<T, kRho, kIn, kOp, kBnd>(a, tile);
    else tile_residual<T, kRho, kIn, kOp, kBnd>(a, tile);
}

template <typename T, bool kRho, int kIn, int kOp, bool kBnd>
__global__ __launch_bounds__(kTileThreads) void k_tile(SweepArgs<T> a) {
    tile_body<T, kRho, kIn, kOp, kBnd>(a, blockIdx.x);
}

// Batched form, as k_sweep_multi (no outflow sides).
template <typename T, bool kRho, int kIn, int kOp>
__global__ __launch_bounds__(kTileThreads) void k_tile_multi(const SweepArgs<T>* __restrict__ descs,
                                                             const int2* __restrict__ tmap) {
    const int2 m = tmap[blockIdx.x];
    const SweepArgs<T> a = descs[m.x];
    tile_body<T, kRho, kIn, kOp, false>(a, m.y);
}

// One problem (a given) or many (d, tmap, tiles).
template <typename T>
struct Launch {
    const SweepArgs<T>* a;
    const SweepArgs<T>* d;
    const int2* tmap;
    int tiles;
    hipStream_t st;
};

template <typename T, bool kRho, int kIn, int kOp>
hipError_t run(const Launch<T>& L) {
    const dim3 grid(L.tiles), block(kTileThreads);
    if (!L.a) hipLaunchKernelGGL((k_tile_multi<T, kRho, kIn, kOp>), grid, block, 0, L.st, L.d, L.tmap);
    else if (L.a->has_bnd) hipLaunchKernelGGL((k_tile<T, kRho, kIn, kOp, true>), grid, block, 0, L.st, *L.a);
    else hipLaunchKernelGGL((k_tile<T, kRho, kIn, kOp, false>), grid, block, 0, L.st, *L.a);
    return hipGetLastError();
}

template <typename T, bool kRho>
hipError_t dispatch(const Launch<T>& L, int in_mode, int op) {
    if (op == kOpResidRestrict) return run<T, kRho, kInPlain, kOpResidRestrict>(L);
    if (op == kOpSweepNorm || op == kOpRefine) {
        if constexpr (sizeof(T) == 8) {
            if (op == kOpSweepNorm) return run<T, kRho, kInPlain, kOpSweepNorm>(L);
            return run<T, kRho, kInCorrect, kOpRefine>(L);
        }
        return hipErrorInvalidValue;
    }
    switch (in_mode) {
        case kInZero: return run<T, kRho, kInZero, kOpSweep>(L);
        case kInPlain: return run<T, kRho, kInPlain, kOpSweep>(L);
        default: return run<T, kRho, kInProlong, kOpSweep>(L);
    }
}

}  // namespace

template <typename T>
hipError_t launch_tile(const SweepArgs<T>& a0, bool use_rho, int in_mode, int op, int* nparts, hipStream_t st) {
    if (!sweep_tileable(a0.nx, a0.ny, a0.nz)) return hipErrorInvalidValue;
    SweepArgs<T> a = a0;
    sweep_geometry(a, kTileCfg);
    const int tiles = sweep_tiles(a.nx, a.ny, a.nz, kTileCfg);
    if (nparts) *nparts = tiles;
    const Launch<T> L{&a, nullptr, nullptr, tiles, st};
    return use_rho ? dispatch<T, true>(L, in_mode, op) : dispatch<T, false>(L, in_mode, op);
}

template <typename T>
hipError_t launch_tile_multi(const SweepArgs<T>* d, const int2* tmap, int tiles, bool use_rho, int in_mode, int op,
                             hipStream_t st) {
    const Launch<T> L{nullptr, d, tmap, tiles, st};
    return use_rho ? dispatch<T, true>(L, in_mode, op) : dispatch<T, false>(L, in_mode, op);
}

template hipError_t launch_tile<double>(const SweepArgs<double>&, bool, int, int, int*, hipStream_t);
template hipError_t launch_tile<float>(const SweepArgs<float>&, bool, int, int, int*, hipStream_t);
template hipError_t launch_tile_multi<double>(const SweepArgs<double>*, const int2*, int, bool, int, int, hipStream_t);
template hipError_t launch_tile_multi<float>(const SweepArgs<float>*, const int2*, int, bool, int, int, hipStream_t);

}  // namespace mg
