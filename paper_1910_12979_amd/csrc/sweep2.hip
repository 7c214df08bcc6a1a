// Two red-black Gauss-Seidel sweeps of a large FP32 level in one launch.
//
// What bounds the FP32 sweep that marches with planes in LDS (sweep.hip) is the
// chain of a plane step, with a barrier in it: fewer instructions or more
// wavefronts changed nothing (256^3 59 us, 47 at the rate of HBM; 512^3 529 and
// 377).  Here a plane step does the four half-sweeps of
// two sweeps, each a plane behind the one before: red of plane t, black of t-1,
// red again of t-2, black again of t-3.  A half-sweep reads in its own plane
// only what the step before wrote, so one barrier a step serves all four.
//
// A wavefront owns 64 columns (one per lane) of an even and an odd row; in a
// plane exactly one of a lane's two cells is red, and in step t it updates its
// row s = (x + t) mod 2 in all four planes.  Values and coefficients are kept
// in registers by colour; neighbours in x come from the lanes beside (no LDS),
// the one in y beyond the pair from the wavefront above or below through LDS
// (one word written and one read a half-sweep).  Coefficients are formed from
// rho once for the two sweeps.  The workgroup covers 56 x 24 cells with a ring of
// four, a chunk of 64 planes marches six more.  256^3 111 us for the two (114
// with the prolongation, 117 from zero; 119, 126 and 118 one by one), 512^3 848,
// 875 and 827 us (1058, 1088 and 967): bound by the issue of about 150 vector
// instructions a step in 16 wavefronts, 1.6 us.
//
// Every cell's expression is the single sweep's, operation by operation, so
// the result is bit for bit that of two of them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "devmath.h"
#include "lanes.h"
#include "mg_internal.h"
#include "sweep2.h"

namespace mg {
namespace {

constexpr int kS2P = 16, kS2TX = kPairTX, kS2TY = kPairTY, kS2TZ = kPairTZ;
static_assert(kS2TX == 64 - 8 && kS2TY == 2 * kS2P - 8, "a ring of four");

template <int kIn>
__global__ __launch_bounds__(64 * kS2P) void k_sweep2(SweepArgs<float> a, int ntx, int nty) {
    constexpr int P = kS2P;
    __shared__ float ex[2][6][P][64];       // B0, R1, B1, R2 (the cells the next step reads), rho rows 0 / 1
    __shared__ float sbc[kS2TZ + 12], sbe[kS2TZ + 12];      // twice beta0, centre / low face, from plane z0 - 4
    const int tile = xcd_order(blockIdx.x, gridDim.x);
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tc = tile / (ntx * nty);
    const int wx = threadIdx.x;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int pd = max(p - 1, 0), pu = min(p + 1, P - 1);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int z0 = tc * kS2TZ, z1 = min(z0 + kS2TZ, nz);
    const int gx = tx * kS2TX - 4 + wx, gy = ty * kS2TY - 4 + 2 * p;
    const int X = fold(gx, nx, 1), Y0 = fold(gy, ny, 1), Y1 = fold(gy + 1, ny, 1);
    const size_t plane = (size_t)nx * ny;
    const unsigned o0 = ((unsigned)Y0 * nx + X) * 4u, o1 = ((unsigned)Y1 * nx + X) * 4u;
    const unsigned oc = ((unsigned)(Y0 >> 1) * (nx >> 1) + (X >> 1)) * 4u;
    const bool xwall = X == 0 && !a.px, ywall0 = Y0 == 0 && !a.py, ywall2 = fold(gy + 2, ny, 1) == 0 && !a.py;
    const bool odd = wx & 1;
    const float h2 = a.h2;
    for (int q = threadIdx.y * 64 + wx; q < z1 - z0 + 10; q += 64 * P) {
        const int k = fold(z0 - 4 + q, nz, 1);
        sbc[q] = (float)(2.0 * a.b0c[k]);
        sbe[q] = (float)(2.0 * a.b0e[k]);
    }
    struct Pair {
        float v0, v1;
    };
    auto ld = [&](const float* __restrict__ g, int k) {
        const float* q = plane_at(g, k, plane);
        return Pair{at_byte(q, o0), at_byte(q, o1)};
    };
    auto ld_phi = [&](int k, float& c) {
        if (kIn == kInProlong) c = at_byte(plane_at(a.phic, k >> 1, plane >> 2), oc);
        return kIn == kInZero ? Pair{0.0f, 0.0f} : ld(a.phi_in, k);
    };
    auto phi_of = [&](Pair v, float c) {
        return kIn == kInProlong ? Pair{v.v0 + c, v.v1 + c} : v;
    };

    // by age: [0] the newest plane a value of its kind exists for
    float B0[3], R1[3], B1[3], R2[3];             // B0: t+1, t, t-1; R1: t, ..; B1: t-1, ..; R2: t-2, ..
    float fR[4], fB[5];                           // t+1, t, ..
    float xR[4], xB[4], lR[4], hR[4], lB[4], hB[4];      // low x, low / high y faces of the red / black cell: t, t-1, ..
    float zR[5], zB[5];                           // low z faces: t+1, t, ..
#pragma unroll
    for (int i = 0; i < 5; ++i) fB[i] = zR[i] = zB[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) fR[i] = xR[i] = xB[i] = lR[i] = hR[i] = lB[i] = hB[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 3; ++i) B0[i] = R1[i] = B1[i] = R2[i] = 0.0f;

    // ahead of the first step, t = z0 - 3 (odd): an even column's red cell is in
    // the odd row there, its black one in the even row
    const int ta = z0 - 3;
    Pair rc;                                      // rho of plane t
    __syncthreads();                              // beta0 staged
    {
        const int k0 = fold(ta, nz, 1), km = fold(ta - 1, nz, 1);
        float c0 = 0.0f, cm = 0.0f;
        const Pair rm = ld(a.rho, km), pm0 = ld_phi(km, cm), pc0 = ld_phi(k0, c0), f0 = ld(a.f, k0);
        rc = ld(a.rho, k0);
        const Pair pm = phi_of(pm0, cm), pc = phi_of(pc0, c0);
        const bool s = !odd;                      // red row of plane t
        const float b = (k0 == 0 && !a.pz) ? 0.0f : 1.0f;
        const float zl0 = pdiv(sbe[1], rm.v0 + rc.v0), zl1 = pdiv(sbe[1], rm.v1 + rc.v1);
        zR[0] = b != 0.0f ? (s ? zl1 : zl0) : 0.0f;
        zB[0] = b != 0.0f ? (s ? zl0 : zl1) : 0.0f;
        fR[0] = s ? f0.v1 : f0.v0;
        fB[0] = s ? f0.v0 : f0.v1;
        B0[0] = s ? pc.v0 : pc.v1;
        B0[1] = s ? pm.v1 : pm.v0;                // plane t-1: the other way round
        ex[0][0][p][wx] = B0[0];
        ex[0][1][p][wx] = ex[0][2][p][wx] = ex[0][3][p][wx] = 0.0f;
        ex[0][4][p][wx] = rc.v0;
        ex[0][5][p][wx] = rc.v1;
    }
    // in flight: phi, rho and f of plane t+1
    int kn = fold(ta + 1, nz, 1);
    float nc = 0.0f;
    Pair np = ld_phi(kn, nc), nr = ld(a.rho, kn), nf = ld(a.f, kn);
    __syncthreads();

    const bool own = wx >= 4 && wx < 60 && p >= 2 && p <= P - 3 && gx < nx;
    const bool own0 = own && gy < ny, own1 = own && gy + 1 < ny;
    int t = ta;
    auto step = [&](auto half) {
        constexpr int h = decltype(half)::value, cur = h, nxt = h ^ 1;
        const bool s = h ? odd : !odd;            // the row updated
        // plane t+1 arrives
        const Pair pn = phi_of(np, nc), rn = nr, fn = nf;
        const int i1 = t + 1 - (z0 - 4);
        const bool zw = kn == 0 && !a.pz;
#pragma unroll
        for (int i = 4; i > 0; --i) {
            fB[i] = fB[i - 1];
            zR[i] = zR[i - 1];
            zB[i] = zB[i - 1];
        }
#pragma unroll
        for (int i = 3; i > 0; --i) {
            fR[i] = fR[i - 1];
            xR[i] = xR[i - 1];
            xB[i] = xB[i - 1];
            lR[i] = lR[i - 1];
            hR[i] = hR[i - 1];
            lB[i] = lB[i - 1];
            hB[i] = hB[i - 1];
        }
#pragma unroll
        for (int i = 2; i > 0; --i) {
            B0[i] = B0[i - 1];
            R1[i] = R1[i - 1];
            B1[i] = B1[i - 1];
            R2[i] = R2[i - 1];
        }
        B0[0] = s ? pn.v1 : pn.v0;
        fR[0] = s ? fn.v0 : fn.v1;
        fB[0] = s ? fn.v1 : fn.v0;
        const float be = sbe[i1], bc = sbc[i1 - 1];
        const float zl0 = zw ? 0.0f : pdiv(be, rc.v0 + rn.v0), zl1 = zw ? 0.0f : pdiv(be, rc.v1 + rn.v1);
        zR[0] = s ? zl0 : zl1;
        zB[0] = s ? zl1 : zl0;
        // plane t+2's loads
        kn = kn + 1 == nz ? 0 : kn + 1;
        np = ld_phi(kn, nc);
        nr = ld(a.rho, kn);
        nf = ld(a.f, kn);
        // what lies beyond the pair
        const int q = s ? pu : pd;
        const float nB0 = ex[cur][0][q][wx], nR1 = ex[cur][1][q][wx], nB1 = ex[cur][2][q][wx],
                    nR2 = ex[cur][3][q][wx];
        const float ru = ex[cur][4][pu][wx], rd = ex[cur][5][pd][wx];
        // coefficients of plane t
        // (the moves between lanes with every lane active, ahead of the choice)
        const float w0 = lane_lo(rc.v0), w1 = lane_lo(rc.v1);
        const float x0 = xwall ? 0.0f : pdiv(bc, w0 + rc.v0), x1 = xwall ? 0.0f : pdiv(bc, w1 + rc.v1);
        const float y0 = ywall0 ? 0.0f : pdiv(bc, rd + rc.v0), ym = pdiv(bc, rc.v0 + rc.v1);
        const float y2 = ywall2 ? 0.0f : pdiv(bc, rc.v1 + ru);
        xR[0] = s ? x1 : x0;
        xB[0] = s ? x0 : x1;
        lR[0] = s ? ym : y0;
        hR[0] = s ? y2 : ym;
        lB[0] = s ? y0 : ym;
        hB[0] = s ? ym : y2;
        rc = rn;
        // one update; xo: the low x face of the lane's other cell (the high one
        // of the cell updated in the lane below), ns: the other cell's value
        auto update = [&](float xl, float xo, float yl, float yh, float zl, float zh, float ns, float outer,
                          float zlo, float zhi, float f) {
            const float xh = lane_hi(xo);
            float num = xl * lane_lo(ns);
            num = num + xh * lane_hi(ns);
            num = num + yl * (s ? ns : outer);
            num = num + yh * (s ? outer : ns);
            num = num + zl * zlo;
            num = num + zh * zhi;
            float den = xl + xh;
            den = den + yl;
            den = den + yh;
            den = den + zl;
            den = den + zh;
            return pdiv(num - h2 * f, den);
        };
        R1[0] = update(xR[0], xB[0], lR[0], hR[0], zR[1], zB[0], B0[1], nB0, B0[2], B0[0], fR[1]);
        B1[0] = update(xB[1], xR[1], lB[1], hB[1], zB[2], zR[1], R1[1], nR1, R1[2], R1[0], fB[2]);
        R2[0] = update(xR[2], xB[2], lR[2], hR[2], zR[3], zB[2], B1[1], nB1, B1[2], B1[0], fR[3]);
        const float B2 = update(xB[3], xR[3], lB[3], hB[3], zB[4], zR[3], R2[1], nR2, R2[2], R2[0], fB[4]);
        ex[nxt][0][p][wx] = B0[0];
        ex[nxt][1][p][wx] = R1[0];
        ex[nxt][2][p][wx] = B1[0];
        ex[nxt][3][p][wx] = R2[0];
        ex[nxt][4][p][wx] = rn.v0;
        ex[nxt][5][p][wx] = rn.v1;
        // the loads are taken up ahead of the stores, so that a wait for them
        // covers the stores of the step before, not these
        at_once(np.v0, np.v1, nr.v0, nr.v1);
        at_once(nf.v0, nf.v1, nc, np.v0);
        const int tb = t - 3;
        if (tb >= z0 && tb < z1) {
            float* o = a.phi_out + (size_t)tb * plane;
            if (own0) put_byte(o, o0, s ? R2[1] : B2);
            if (own1) put_byte(o, o1, s ? B2 : R2[1]);
        }
        ++t;
        __syncthreads();
    };
    while (t <= z1 + 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
}

}  // namespace

bool sweep_paired(int nx, int ny, int nz) {
    if (!sweep_marchable(nx, ny, nz) || tune_forced() >= 0) return false;
    const double blocks = (double)((nx + kPairTX - 1) / kPairTX) * ((ny + kPairTY - 1) / kPairTY) *
                          ((nz + kPairTZ - 1) / kPairTZ);
    const double rounds = std::ceil(blocks / 256.0), steps = std::min(nz, kPairTZ) + 6;
    return rounds * steps * 1.65 < 2.0 * 3.52e-6 * ((double)nx * ny * nz);
}

hipError_t launch_sweep2(const SweepArgs<float>& a, int in_mode, hipStream_t st) {
    const int ntx = (a.nx + kS2TX - 1) / kS2TX, nty = (a.ny + kS2TY - 1) / kS2TY, nch = (a.nz + kS2TZ - 1) / kS2TZ;
    const dim3 grid(ntx * nty * nch), block(64, kS2P);
    if (in_mode == kInZero) hipLaunchKernelGGL(k_sweep2<kInZero>, grid, block, 0, st, a, ntx, nty);
    else if (in_mode == kInPlain) hipLaunchKernelGGL(k_sweep2<kInPlain>, grid, block, 0, st, a, ntx, nty);
    else hipLaunchKernelGGL(k_sweep2<kInProlong>, grid, block, 0, st, a, ntx, nty);
    return hipGetLastError();
}

}  // namespace mg
