// Nodal levels and the kernels that march up through their planes.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "devmath.h"
#include "lanes.h"
#include "mg_internal.h"

namespace mg {
namespace {

// One level of the nodal hierarchy: cells (nx, ny, nz), nodes (Nx, Ny, Nz);
// arrays in T (FP64, or FP32 for the inner cycle of a mixed-precision solve).
template <typename T>
struct NodLevelT {
    int nx, ny, nz;
    int Nx, Ny, Nz;
    int px, py, pz;
    double h;
    T* sig;             // cells
    T* phi;             // nodes
    T* f;
    T* phi2;            // nodes: the other buffer of the out-of-place fused sweep
    __host__ __device__ size_t nodes() const { return (size_t)Nx * Ny * Nz; }
    __host__ __device__ size_t cells() const { return (size_t)nx * ny * nz; }
};
using NodLevel = NodLevelT<double>;

// A cell coefficient as a node column uses it: of the cell on its high side
// in x (the lane's own) and on its low side (the lane's below).
template <typename T>
struct SigPair {
    T hi, lo;
};
template <typename T>
__device__ __forceinline__ SigPair<T> sig_pair(T s) {
    return SigPair<T>{s, lane_lo(s)};
}

// Values of one column in the planes below, at and above a node.
template <typename T>
struct Col3 {
    T b, c, t;
};

// A node's Gauss-Seidel update (num - c12 f) / den, num = sum_cells sigma
// (far corners), den = 4 sum_cells sigma, from the columns of phi at x in the
// rows below (dn) and above (up) and in the node's own row (ob, ot: the
// planes below and above), and the cells' coefficients by row (l: below,
// u: above) and layer (b, t).  Of the four far corners of a cell on the high
// side in x, three lie in the column x + 1 and one (y and z moved) in the
// node's own: a lane forms the three-corner sums q of its own column once,
// weights them with the cells on either side and hands the two results to
// the lanes beside it, so that a node's 20 neighbours and 8 cells cost 8
// values of phi and 4 of sigma per lane.
template <typename T>
__device__ __forceinline__ T nod_update(const Col3<T>& dn, const Col3<T>& up, T ob, T ot, const SigPair<T>& lb,
                                        const SigPair<T>& ub, const SigPair<T>& lt, const SigPair<T>& ut, T c12,
                                        T f) {
    const T q00 = (dn.c + ob) + dn.b, q10 = (up.c + ob) + up.b;
    const T q01 = (dn.c + ot) + dn.t, q11 = (up.c + ot) + up.t;
    const T toLo = fma(ut.lo, q11, fma(lt.lo, q01, fma(ub.lo, q10, lb.lo * q00)));   // for the node at x - 1
    const T toHi = fma(ut.hi, q11, fma(lt.hi, q01, fma(ub.hi, q10, lb.hi * q00)));   // for the node at x + 1
    const T s00 = lb.lo + lb.hi, s10 = ub.lo + ub.hi, s01 = lt.lo + lt.hi, s11 = ut.lo + ut.hi;
    const T own = fma(s11, up.t, fma(s01, dn.t, fma(s10, up.b, s00 * dn.b)));
    const T den = T(4) * ((s00 + s10) + (s01 + s11));
    const T num = own + (lane_hi(toLo) + lane_lo(toHi));
    return pdiv(fma(-c12, f, num), den);
}

// ---------------------------------------------------------------------------
// Fused out-of-place sweep: out = the four-colour Gauss-Seidel sweep of
// L.phi (colours 0..3 in order), one launch.
//
// Colour c of node (I, J, K) is (J mod 2) + 2 (K mod 2); every row of nodes
// along x has one colour.  Coupled nodes differ in at least two coordinates,
// so in an even plane colour 0 reads only old values and colour 1 the new
// colour-0 values of its four in-plane diagonal neighbours (old values
// above and below); in an odd plane colour 2 reads the new values of the
// even planes above and below, colour 3 those and the new colour-2 values of
// its in-plane diagonal neighbours.
//
// A workgroup owns a tile of 56 x (2P - 8) nodes and a chunk of planes and
// marches up through it, one even plane and the odd plane below it per step:
// colour 0 of the even plane on the tile plus a ring of 3, colour 1 on ring
// 2, then colour 2 of the odd plane on ring 1 and colour 3 on the tile, so
// every value a later colour reads was computed by the workgroup itself;
// loads cover the tile plus a ring of 4: 64 columns, one per lane, and 2P
// rows, an even and an odd one per wavefront.  The even plane at the top of
// a chunk is computed again by the next chunk (it reads only old values).
// Cells beyond a wall carry sigma = 0 and nodes beyond it the value 0, so
// their terms add exact zeros.
//
// A lane keeps its two rows of phi (four planes), sigma (three layers) and f
// in registers and takes what lies beside it from the lanes beside it; only
// the row above or below the pair comes through LDS (3 reads an update).  A
// step has four barriers; the loads of the next one are in flight meanwhile.
// A large sweep is bound by the issue of FP64 instructions (about 40 of 5
// cycles an update, 1.7 updates a node at 256^3 with the halo) and by reading
// phi, sigma and f through the caches 1.5 to 1.7 times: 256^3 nodes 144 us
// (204 with 28 values of LDS an update, every neighbour read there), 128^3
// 26 us (50 with a launch per colour), 64^3 9.4 us (17); FP32 256^3 65 us.
// An XCD's workgroups take consecutive tiles, so that most of what their
// windows share is in its L2 (128^3: 40 us without, 192^3 69 / 102).
// kProlong: phi is read with the correction of the coarser level C added,
// phi + P C.phi (P trilinear), so the prolongation needs no pass of its own
// (256^3: 170 us for the sweep with it against 144 + 63).
// ---------------------------------------------------------------------------
constexpr int kNodTX = 56;

template <typename T, int P, bool kProlong>
__global__ __launch_bounds__(64 * P) void k_nod_sweep(NodLevelT<T> L, T* __restrict__ out, int tz, int ntx, int nty,
                                                      int etop, NodLevelT<T> C) {
    constexpr int TY = 2 * P - 8;
    __shared__ T se[4][P][64];              // even rows of a plane, by (plane - ks) & 3
    __shared__ T so[4][P][64];              // odd rows
    __shared__ T sc[2][P][64];              // odd rows of the two newest cell layers
    const int tile = xcd_order(blockIdx.x, gridDim.x);
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tc = tile / (ntx * nty);
    const int ks = tc * tz, ke = min(ks + tz, etop);
    const int wx = threadIdx.x;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int pd = max(p - 1, 0), pu = min(p + 1, P - 1);
    // global node / low-corner cell coordinates of the column and of its two rows
    const int gI = tx * kNodTX - 4 + wx, gJe = ty * TY - 4 + 2 * p, gJo = gJe + 1;
    auto in = [](int g, int n, int per) { return per || (g >= 0 && g < n); };
    const bool xn = in(gI, L.Nx, L.px), xc = in(gI, L.nx, L.px);
    const bool yne = in(gJe, L.Ny, L.py), yce = in(gJe, L.ny, L.py);
    const bool yno = in(gJo, L.Ny, L.py), yco = in(gJo, L.ny, L.py);
    const int Iw = fold(gI, L.Nx, L.px), iw = fold(gI, L.nx, L.px);
    const int Je = fold(gJe, L.Ny, L.py), Jo = fold(gJo, L.Ny, L.py);
    const int je = fold(gJe, L.ny, L.py), jo = fold(gJo, L.ny, L.py);
    const size_t NxNy = (size_t)L.Nx * L.Ny, nxny = (size_t)L.nx * L.ny;
    constexpr unsigned kB = sizeof(T);            // byte offsets within a plane
    const unsigned ne = ((unsigned)Je * L.Nx + Iw) * kB, no = ((unsigned)Jo * L.Nx + Iw) * kB;
    const unsigned ce = ((unsigned)je * L.nx + iw) * kB, co = ((unsigned)jo * L.nx + iw) * kB;
    const T c12 = (T)(12.0 * (L.h * L.h));
    auto plane_ok = [&](int K) { return in(K, L.Nz, L.pz); };
    auto layer_ok = [&](int k) { return in(k, L.nz, L.pz); };
    // Loads are always issued from valid (wrapped or clamped) addresses; cells
    // beyond a wall become 0 when they are taken up (so the clamped values of
    // nodes beyond it, which are never updated, add exact zeros).
    auto ld_node = [&](const T* __restrict__ a, int K, T& e, T& o) {      // K, k: folded
        const T* q = plane_at(a, K, NxNy);
        e = at_byte(q, ne);
        o = at_byte(q, no);
    };
    auto ld_sig = [&](int k, T& e, T& o) {
        const T* q = plane_at(L.sig, k, nxny);
        e = at_byte(q, ce);
        o = at_byte(q, co);
    };
    auto fn = [&](int K) { return fold(K, L.Nz, L.pz); };
    auto fc = [&](int k) { return fold(k, L.nz, L.pz); };
    // The coarse correction: an even column reads its parent, an odd one the
    // parent above it and takes the other from the lane below; in the coarse
    // rows at and above the even row.
    const bool oddx = wx & 1;
    unsigned c0 = 0, c1 = 0;
    if (kProlong) {
        const int I1 = fold((Iw + 1) >> 1, C.Nx, L.px);
        const int J0 = Je >> 1, J1 = fold((Jo + 1) >> 1, C.Ny, L.py);
        c0 = ((unsigned)J0 * C.Nx + I1) * kB;
        c1 = ((unsigned)J1 * C.Nx + I1) * kB;
    }
    auto ld_coarse = [&](int K, T& a, T& b) {     // K: coarse plane, folded
        const T* q = plane_at(C.phi, K, (size_t)C.Nx * C.Ny);
        a = at_byte(q, c0);
        b = at_byte(q, c1);
    };
    // its values in the even (e) and the odd row (o)
    auto interp = [&](T a, T b, T& e, T& o) {
        const T al = lane_lo(a), bl = lane_lo(b);
        e = oddx ? T(0.5) * (al + a) : a;
        o = T(0.5) * (e + (oddx ? T(0.5) * (bl + b) : b));
    };

    // phi, rows e / o, of planes E-2 .. E+1 and sigma, rows e-1 / e / o, of
    // layers E-2 .. E: entry (i + 2 h) mod 4 and i (h = 0) or 2 - i (h = 1) of
    // step h = E / 2 mod 2, so that a step overwrites what the next one no
    // longer needs and moves nothing.
    T pe[4], po[4];
    SigPair<T> sm[3], s0[3], s1[3];
    T fe0, fo0, fe1 = T(0), fo1 = T(0);           // f of plane E, of the plane below
    T ge = T(0), go = T(0);                       // coarse correction in plane E + 2
    auto maskc = [&](T v, bool y, bool z) { return (xc && y && z) ? v : T(0); };
    pe[0] = po[0] = T(0);
    sm[0] = s0[0] = s1[0] = SigPair<T>{T(0), T(0)};
    ld_node(L.phi, fn(ks - 1), pe[1], po[1]);
    ld_node(L.phi, fn(ks), pe[2], po[2]);
    ld_node(L.phi, fn(ks + 1), pe[3], po[3]);
    {
        T a3, b3, a4, b4;
        ld_sig(fc(ks - 1), a3, b3);
        ld_sig(fc(ks), a4, b4);
        ld_node(L.f, fn(ks), fe0, fo0);
        if (kProlong) {
            T ue, uo, ve, vo, we, wo;
            ld_coarse(fold((ks - 2) / 2, C.Nz, L.pz), ue, uo);
            ld_coarse(fold(ks / 2, C.Nz, L.pz), ve, vo);
            ld_coarse(fold((ks + 2) / 2, C.Nz, L.pz), we, wo);
            interp(ue, uo, ue, uo);
            interp(ve, vo, ve, vo);
            interp(we, wo, we, wo);
            pe[1] += T(0.5) * (ue + ve);
            po[1] += T(0.5) * (uo + vo);
            pe[2] += ve;
            po[2] += vo;
            pe[3] += T(0.5) * (ve + we);
            po[3] += T(0.5) * (vo + wo);
            ge = we;
            go = wo;
        }
        s0[1] = sig_pair(maskc(a3, yce, layer_ok(ks - 1)));
        s1[1] = sig_pair(maskc(b3, yco, layer_ok(ks - 1)));
        s0[2] = sig_pair(maskc(a4, yce, layer_ok(ks)));
        s1[2] = sig_pair(maskc(b4, yco, layer_ok(ks)));
    }
    so[3][p][wx] = po[1];                         // plane K in entry (K - ks) mod 4
    so[0][p][wx] = po[2];
    so[1][p][wx] = po[3];
    se[3][p][wx] = pe[1];
    sc[0][p][wx] = s1[1].hi;
    sc[1][p][wx] = s1[2].hi;
    __syncthreads();

    // output nodes (unwrapped inside the box)
    const bool tile_pair = wx >= 4 && wx < 60 && gI < L.Nx;
    const bool oute = tile_pair && gJe < L.Ny, outo = tile_pair && gJo < L.Ny;
    const bool rows_out = p >= 2 && p <= P - 3;
    // planes E+1, E+2, E+3 and layers E+1, E+2, folded; two on per step (at
    // least two planes and two layers in a periodic direction)
    int k1 = fn(ks + 1), k2 = fn(ks + 2), k3 = fn(ks + 3), l1 = fc(ks + 1), l2 = fc(ks + 2);
    int kc = kProlong ? fold(ks / 2 + 2, C.Nz, L.pz) : 0;
    int ko0 = fn(ks), ko1 = fn(ks - 1);           // planes E and E-1
    auto on = [&](int& k, int step, int n) {
        k += step;
        if (L.pz) k = k >= n ? k - n : k;
        else k = min(k, n - 1);
    };
    int E = ks;
    auto step = [&](auto half) -> bool {
        constexpr int h = decltype(half)::value;
        constexpr int i0 = 2 * h, i1 = 2 * h + 1, i2 = 2 - 2 * h, i3 = 3 - 2 * h;      // planes E-2 .. E+1
        constexpr int l0 = 2 * h, lm = 1, lt = 2 - 2 * h;                              // layers E-2, E-1, E
        constexpr int tm2 = (2 * h + 2) & 3, tm1 = (2 * h + 3) & 3, t0 = 2 * h, t1 = 2 * h + 1;
        const bool more = E + 2 <= ke;
        // the next step's loads: planes E+2, E+3, layers E+1, E+2, f of planes E+2, E+1
        T q0, q1, q2, q3, r0, r1, r2, r3, nfe, nfo, nfe1, nfo1;
        ld_node(L.phi, k2, q0, q1);
        ld_node(L.phi, k3, q2, q3);
        ld_sig(l1, r0, r1);
        ld_sig(l2, r2, r3);
        ld_node(L.f, k2, nfe, nfo);
        ld_node(L.f, k1, nfe1, nfo1);
        T qa = T(0), qb = T(0);
        if (kProlong) ld_coarse(kc, qa, qb);
        sm[lm] = sig_pair(sc[0][pd][wx]);
        sm[lt] = sig_pair(sc[1][pd][wx]);
        const bool even_ok = plane_ok(E);
        // A: colour 0 of plane E (ring 3)
        if (p >= 1) {
            const Col3<T> dn{so[tm1][pd][wx], so[t0][pd][wx], so[t1][pd][wx]};
            const Col3<T> up{po[i1], po[i2], po[i3]};
            const T v = nod_update(dn, up, pe[i1], pe[i3], sm[lm], s0[lm], sm[lt], s0[lt], c12, fe0);
            if (xn && yne && even_ok) pe[i2] = v;
        }
        se[t0][p][wx] = pe[i2];
        se[t1][p][wx] = pe[i3];
        __syncthreads();
        // B: colour 1 of plane E (ring 2)
        if (p >= 1 && p <= P - 2) {
            const Col3<T> dn{pe[i1], pe[i2], pe[i3]};
            const Col3<T> up{se[tm1][pu][wx], se[t0][pu][wx], se[t1][pu][wx]};
            const T v = nod_update(dn, up, po[i1], po[i3], s0[lm], s1[lm], s0[lt], s1[lt], c12, fo0);
            if (xn && yno && even_ok) po[i2] = v;
            so[t0][p][wx] = po[i2];
        }
        __syncthreads();
        T vo1 = T(0);
        if (E > ks) {
            // C: colour 2 of plane E-1 (ring 1)
            if (p >= 2 && p <= P - 2) {
                const Col3<T> dn{so[tm2][pd][wx], so[tm1][pd][wx], so[t0][pd][wx]};
                const Col3<T> up{po[i0], po[i1], po[i2]};
                const T v = nod_update(dn, up, pe[i0], pe[i2], sm[l0], s0[l0], sm[lm], s0[lm], c12, fe1);
                if (xn && yne) pe[i1] = v;
                se[tm1][p][wx] = pe[i1];
            }
            __syncthreads();
            // D: colour 3 of plane E-1 (tile)
            if (rows_out) {
                const Col3<T> dn{pe[i0], pe[i1], pe[i2]};
                const Col3<T> up{se[tm2][pu][wx], se[tm1][pu][wx], se[t0][pu][wx]};
                vo1 = nod_update(dn, up, po[i0], po[i2], s0[l0], s1[l0], s0[lm], s1[lm], c12, fo1);
            }
        }
        // The loads are taken up here, ahead of this step's stores: a wait for
        // them then covers the stores of the step before, not these.
        at_once(q0, q1, q2, q3);
        at_once(r0, r1, r2, r3);
        at_once(nfe, nfo, nfe1, nfo1);
        if (kProlong) at_once(qa, qb, q0, q1);
        // planes E (where this chunk owns it) and E-1 written
        if (rows_out) {
            if (even_ok && (E < ke || (!L.pz && ke == etop))) {
                T* q = out + (size_t)(unsigned)ko0 * NxNy;
                if (oute) put_byte(q, ne, pe[i2]);
                if (outo) put_byte(q, no, po[i2]);
            }
            if (E > ks) {
                T* q = out + (size_t)(unsigned)ko1 * NxNy;
                if (oute) put_byte(q, ne, pe[i1]);
                if (outo) put_byte(q, no, vo1);
            }
        }
        if (!more) return false;
        if (kProlong) {
            T we, wo;
            interp(qa, qb, we, wo);
            q0 += ge;
            q1 += go;
            q2 += T(0.5) * (ge + we);
            q3 += T(0.5) * (go + wo);
            ge = we;
            go = wo;
            on(kc, 1, C.Nz);
        }
        const bool okl1 = layer_ok(E + 1), okl2 = layer_ok(E + 2);
        pe[i0] = q0;
        po[i0] = q1;
        pe[i1] = q2;
        po[i1] = q3;
        s0[lm] = sig_pair(maskc(r0, yce, okl1));
        s1[lm] = sig_pair(maskc(r1, yco, okl1));
        s0[l0] = sig_pair(maskc(r2, yce, okl2));
        s1[l0] = sig_pair(maskc(r3, yco, okl2));
        // the odd rows of planes E-2, E-1 and layers E-1, E were last read
        // before the barrier ahead of D (in the first step, of B)
        so[tm2][p][wx] = po[i0];
        so[tm1][p][wx] = po[i1];
        sc[0][p][wx] = s1[lm].hi;
        sc[1][p][wx] = s1[l0].hi;
        fe0 = nfe;
        fo0 = nfo;
        fe1 = nfe1;
        fo1 = nfo1;
        ko1 = k1;
        ko0 = k2;
        on(k1, 2, L.Nz);
        on(k2, 2, L.Nz);
        on(k3, 2, L.Nz);
        on(l1, 2, L.nz);
        on(l2, 2, L.nz);
        E += 2;
        __syncthreads();
        return true;
    };
    while (step(std::integral_constant<int, 0>{}) && step(std::integral_constant<int, 1>{})) {
    }
}

// ---------------------------------------------------------------------------
// Residual r = f - L phi, (L phi)_n = 1/(12 h^2) sum_c sigma_c (far corners -
// 4 phi_n), by wavefronts that each march up through a chunk of planes with
// 64 columns of four rows: phi of three planes (six rows) and sigma of two
// layers (five rows) in registers, what lies beside a column from the lanes
// beside it as in nod_update, the next plane's loads in flight.  What bounds
// it is reading phi, sigma and f once: 256^3 nodes in FP64 94 us with the norm
// (4.3 TB/s; 150 from tiles staged in LDS), 122 us with the restriction (218 in
// two kernels with r in memory between them), 171 us with the refinement.  The
// far corners enter as differences from phi_n, formed before the sum.
//
// kRestrict: full weighting of r in the same pass, coarse f = 1/8 sum_d
// prod(1 - |d_i|/2) r_{2C+d} and coarse phi = 0; r itself is not written.  The
// row of r below a wavefront's comes from the wavefront below through LDS (a
// workgroup's lowest wavefront serves only that and one coarse row).
// kNorm: the workgroup's partial row {sum r^2, 0, max |r|, #non-finite} at row
// blockIdx.x.  kRefine: the refinement step of a mixed-precision solve as
// well: phi is phi + corr / s (corr the FP32 V-cycle's correction, s =
// scales[0] the scale its residual carried, a power of two), written out of
// place, and the residual of the updated phi is written in FP32 times
// scales[1] (the scale of the previous residual: lagged by one step, as the
// reduction advances the scales afterwards).
// ---------------------------------------------------------------------------
struct NodRefine {
    const float* corr;
    const double* scales;
    double* phi_out;
    float* r32;
};
enum NodResidMode { kNodRestrict, kNodNorm, kNodRefine };

// Difference form of a node's sum: sum_c sigma_c (far corners - 4 pn).
template <typename T>
__device__ __forceinline__ T nod_flux(const Col3<T>& dn, const Col3<T>& up, T ob, T pn, T ot, T pn3_lo, T pn3_hi,
                                      const SigPair<T>& lb, const SigPair<T>& ub, const SigPair<T>& lt,
                                      const SigPair<T>& ut) {
    const T q00 = (dn.c + ob) + dn.b, q10 = (up.c + ob) + up.b;
    const T q01 = (dn.c + ot) + dn.t, q11 = (up.c + ot) + up.t;
    const T toLo = fma(ut.lo, q11 - pn3_lo,
                       fma(lt.lo, q01 - pn3_lo, fma(ub.lo, q10 - pn3_lo, lb.lo * (q00 - pn3_lo))));
    const T toHi = fma(ut.hi, q11 - pn3_hi,
                       fma(lt.hi, q01 - pn3_hi, fma(ub.hi, q10 - pn3_hi, lb.hi * (q00 - pn3_hi))));
    const T s00 = lb.lo + lb.hi, s10 = ub.lo + ub.hi, s01 = lt.lo + lt.hi, s11 = ut.lo + ut.hi;
    const T own = fma(s11, up.t - pn, fma(s01, dn.t - pn, fma(s10, up.b - pn, s00 * (dn.b - pn))));
    return own + (lane_hi(toLo) + lane_lo(toHi));
}

constexpr int kNodResidRows = 4;                  // rows of a wavefront
// Four wavefronts: with eight the restriction of 256^3 nodes took 125 us
// against 122, the norm 99 against 94 (barriers over more wavefronts, and two
// workgroups of them do not fill a SIMD's registers).
constexpr int kNodResidWaves = 4;
// columns and rows of a workgroup's tile, in fine nodes
inline __host__ __device__ int nod_resid_tx(bool restr) { return restr ? 60 : 62; }
inline __host__ __device__ int nod_resid_ty(bool restr) {
    return restr ? 2 * (2 * kNodResidWaves - 1) : kNodResidRows * kNodResidWaves;
}

template <typename T, int kMode>
__global__ __launch_bounds__(64 * kNodResidWaves) void k_nod_resid(NodLevelT<T> L, NodLevelT<T> C, int tz, int ntx, int nty,
                                                      double* __restrict__ partials, NodRefine ra) {
    constexpr bool kRestrict = kMode == kNodRestrict, kRefine = kMode == kNodRefine;
    constexpr int R = kNodResidRows, P = kNodResidWaves;
    __shared__ double sh[kRestrict ? 2 * P * 64 : 3 * P];
    const int tile = xcd_order(blockIdx.x, gridDim.x);
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tc = tile / (ntx * nty);
    const int wx = threadIdx.x;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int gI = tx * nod_resid_tx(kRestrict) - (kRestrict ? 2 : 1) + wx;
    const int gJ = ty * nod_resid_ty(kRestrict) - (kRestrict ? 2 : 0) + R * p;      // first of the four rows
    // fine planes: [Ka, Kb); restricting, of coarse planes [tc tz, ..): one plane below the first to one above the last
    const int Ka = kRestrict ? 2 * tc * tz - 1 : tc * tz;
    const int Kb = kRestrict ? 2 * min(tc * tz + tz, C.Nz) : min(Ka + tz, L.Nz);
    auto in = [](int g, int n, int per) { return per || (g >= 0 && g < n); };
    const size_t NxNy = (size_t)L.Nx * L.Ny, nxny = (size_t)L.nx * L.ny;
    const bool xn = in(gI, L.Nx, L.px), xc = in(gI, L.nx, L.px);
    constexpr unsigned kB = sizeof(T);
    const unsigned xo = (unsigned)fold(gI, L.Nx, L.px), co = (unsigned)fold(gI, L.nx, L.px) * kB;
    size_t nrow[R + 2], crow[R + 1];              // rows gJ - 1 .. gJ + 4 of nodes, gJ - 1 .. gJ + 3 of cells
    bool cok[R + 1];
#pragma unroll
    for (int j = 0; j < R + 2; ++j) nrow[j] = (size_t)fold(gJ - 1 + j, L.Ny, L.py) * L.Nx;
#pragma unroll
    for (int j = 0; j < R + 1; ++j) {
        crow[j] = (size_t)fold(gJ - 1 + j, L.ny, L.py) * L.nx;
        cok[j] = xc && in(gJ - 1 + j, L.ny, L.py);
    }
    const double inv_s = kRefine ? 1.0 / ra.scales[0] : 0.0;     // exact: a power of two
    const double r_s = kRefine ? ra.scales[1] : 0.0;
    const T ih = (T)(12.0 * L.h * L.h);

    auto ld_phi = [&](int K, T (&v)[R + 2], float (&c)[R + 2]) {
        const T* q = plane_at(L.phi, K, NxNy);
#pragma unroll
        for (int j = 0; j < R + 2; ++j) v[j] = at_byte(q + nrow[j], xo * kB);
        if (kRefine) {
            const float* d = plane_at(ra.corr, K, NxNy);
#pragma unroll
            for (int j = 0; j < R + 2; ++j) c[j] = at_byte(d + nrow[j], xo * 4u);
        }
    };
    auto ld_sig = [&](int k, T (&v)[R + 1]) {
        const T* q = plane_at(L.sig, k, nxny);
#pragma unroll
        for (int j = 0; j < R + 1; ++j) v[j] = at_byte(q + crow[j], co);
    };
    auto ld_f = [&](int K, T (&v)[R]) {
        const T* q = plane_at(L.f, K, NxNy);
#pragma unroll
        for (int j = 0; j < R; ++j) v[j] = at_byte(q + nrow[j + 1], xo * kB);
    };
    // phi of a plane as the residual takes it
    auto take = [&](T (&v)[R + 2], const T (&q)[R + 2], const float (&c)[R + 2]) {
#pragma unroll
        for (int j = 0; j < R + 2; ++j) v[j] = kRefine ? (T)(q[j] + (double)c[j] * inv_s) : q[j];
    };
    auto take_sig = [&](SigPair<T> (&v)[R + 1], const T (&q)[R + 1], bool ok) {
#pragma unroll
        for (int j = 0; j < R + 1; ++j) v[j] = sig_pair((ok && cok[j]) ? q[j] : T(0));
    };
    auto fn = [&](int K) { return fold(K, L.Nz, L.pz); };
    auto fc = [&](int k) { return fold(k, L.nz, L.pz); };

    T pb[R + 2], pc[R + 2], pt[R + 2], f[R];      // planes K-1, K, K+1
    SigPair<T> sb[R + 1], st[R + 1];              // layers K-1, K
    {
        T v0[R + 2], v1[R + 2], v2[R + 2], s0[R + 1], s1[R + 1];
        float c0[R + 2] = {}, c1[R + 2] = {}, c2[R + 2] = {};
        ld_phi(fn(Ka - 1), v0, c0);
        ld_phi(fn(Ka), v1, c1);
        ld_phi(fn(Ka + 1), v2, c2);
        ld_sig(fc(Ka - 1), s0);
        ld_sig(fc(Ka), s1);
        ld_f(fn(Ka), f);
        take(pb, v0, c0);
        take(pc, v1, c1);
        take(pt, v2, c2);
        take_sig(sb, s0, in(Ka - 1, L.nz, L.pz));
        take_sig(st, s1, in(Ka, L.nz, L.pz));
    }
    int k0 = fn(Ka), k1 = fn(Ka + 1), k2 = fn(Ka + 2), l1 = fc(Ka + 1);
    auto on = [&](int& k, int K, int n) {         // k, the fold of plane or layer K - 1, to that of K
        ++k;
        if (L.pz) k = k >= n ? 0 : k;
        else k = min(max(K, 0), n - 1);
    };
    double s2 = 0.0, mx = 0.0, nonfin = 0.0;
    T acc0 = T(0), acc1 = T(0);                   // restriction: planes so far of the two coarse rows
    for (int K = Ka; K < Kb; ++K) {
        T q[R + 2], qs[R + 1], qf[R];
        float qc[R + 2] = {};
        ld_phi(k2, q, qc);
        ld_sig(l1, qs);
        ld_f(k1, qf);
        T r[R];
        const bool zok = in(K, L.Nz, L.pz);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const T pn = pc[j + 1], pn3 = T(3) * pn;
            const T sum = nod_flux(Col3<T>{pb[j], pc[j], pt[j]}, Col3<T>{pb[j + 2], pc[j + 2], pt[j + 2]}, pb[j + 1],
                                   pn, pt[j + 1], lane_lo(pn3), lane_hi(pn3), sb[j], sb[j + 1], st[j], st[j + 1]);
            const bool ok = zok && xn && in(gJ + j, L.Ny, L.py);
            r[j] = ok ? f[j] - pdiv(sum, ih) : T(0);
        }
        if (kRestrict) {
            T* row = reinterpret_cast<T*>(sh) + (K & 1) * (P * 64);
            row[p * 64 + wx] = r[3];
            __syncthreads();
            const T below = row[max(p - 1, 0) * 64 + wx];
            const T a = r[0] + T(0.5) * (below + r[1]), b = r[2] + T(0.5) * (r[1] + r[3]);
            const T wa = a + T(0.5) * (lane_lo(a) + lane_hi(a)), wb = b + T(0.5) * (lane_lo(b) + lane_hi(b));
            if (K & 1) {
                acc0 = fma(T(0.5), wa, acc0);
                acc1 = fma(T(0.5), wb, acc1);
                if (K > Ka) {
                    // coarse plane (K - 1) / 2 is complete
                    const int I = gI >> 1, J = gJ >> 1;          // coarse node; gI even on the lanes that write
                    T* cf = C.f + (size_t)((K - 1) / 2) * ((size_t)C.Nx * C.Ny);
                    T* cp = C.phi + (size_t)((K - 1) / 2) * ((size_t)C.Nx * C.Ny);
                    const bool own = !(wx & 1) && wx >= 2 && wx <= 60 && I < C.Nx;
                    if (own && p > 0 && J < C.Ny) {
                        cf[(size_t)J * C.Nx + I] = T(0.125) * acc0;
                        cp[(size_t)J * C.Nx + I] = T(0);
                    }
                    if (own && J + 1 < C.Ny) {
                        cf[(size_t)(J + 1) * C.Nx + I] = T(0.125) * acc1;
                        cp[(size_t)(J + 1) * C.Nx + I] = T(0);
                    }
                }
                acc0 = T(0.5) * wa;
                acc1 = T(0.5) * wb;
            } else {
                acc0 += wa;
                acc1 += wb;
            }
        } else {
            const bool own = wx >= 1 && wx <= 62 && gI < L.Nx;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (!own || gJ + j >= L.Ny) continue;
                const double rd = (double)r[j];
                if (!isfinite(rd)) nonfin += 1.0;
                s2 += rd * rd;
                mx = fmax(mx, fabs(rd));
                if (kRefine) {
                    const size_t n = (size_t)k0 * NxNy + nrow[j + 1] + xo;
                    ra.phi_out[n] = pc[j + 1];
                    ra.r32[n] = (float)(r[j] * r_s);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < R + 2; ++j) {
            pb[j] = pc[j];
            pc[j] = pt[j];
        }
        take(pt, q, qc);
#pragma unroll
        for (int j = 0; j < R + 1; ++j) sb[j] = st[j];
        take_sig(st, qs, in(K + 1, L.nz, L.pz));
#pragma unroll
        for (int j = 0; j < R; ++j) f[j] = qf[j];
        k0 = k1;
        k1 = k2;
        on(k2, K + 3, L.Nz);
        on(l1, K + 2, L.nz);
    }
    if (!kRestrict) {
        // fixed-order trees over the wavefront, then over the workgroup
        for (int w = 32; w > 0; w >>= 1) {
            s2 = s2 + __shfl_down(s2, w);
            mx = fmax(mx, __shfl_down(mx, w));
            nonfin = nonfin + __shfl_down(nonfin, w);
        }
        if (wx == 0) {
            sh[3 * p] = s2;
            sh[3 * p + 1] = mx;
            sh[3 * p + 2] = nonfin;
        }
        __syncthreads();
        if (wx == 0 && p == 0) {
            for (int w = 1; w < P; ++w) {
                s2 = s2 + sh[3 * w];
                mx = fmax(mx, sh[3 * w + 1]);
                nonfin = nonfin + sh[3 * w + 2];
            }
            double* row = partials + (size_t)blockIdx.x * kReduceWidth;
            row[0] = s2;
            row[1] = 0.0;
            row[2] = mx;
            row[3] = nonfin;
        }
    }
}

// Levels whose colouring is consistent across periodic wraps (even node
// counts there), with an even number of node planes to march (the top plane
// of a walled z is even).
template <typename T>
bool nod_sweep_fits(const NodLevelT<T>& L) {
    if (L.py && L.Ny % 2 != 0) return false;
    if (L.pz ? (L.Nz % 2 != 0) : (L.nz % 2 != 0)) return false;
    return (L.pz ? L.Nz : L.Nz - 1) >= 2;
}

template <typename T, int P>
hipError_t launch_nod_sweep_t(const NodLevelT<T>& L, T* out, int tz, const NodLevelT<T>* coarse, hipStream_t st) {
    const int etop = L.pz ? L.Nz : L.Nz - 1, ty = 2 * P - 8;
    const int ntx = (L.Nx + kNodTX - 1) / kNodTX, nty = (L.Ny + ty - 1) / ty, nch = (etop + tz - 1) / tz;
    const dim3 grid(ntx * nty * nch), block(64, P);
    if (coarse)
        hipLaunchKernelGGL((k_nod_sweep<T, P, true>), grid, block, 0, st, L, out, tz, ntx, nty, etop, *coarse);
    else
        hipLaunchKernelGGL((k_nod_sweep<T, P, false>), grid, block, 0, st, L, out, tz, ntx, nty, etop, L);
    return hipGetLastError();
}

// Workgroups of the residual on a level, in chunks of tz planes (restricting,
// of coarse planes).
struct NodResidGrid {
    int tz, ntx, nty, nch;
    int blocks() const { return ntx * nty * nch; }
};
inline NodResidGrid nod_resid_grid_of(int Nx, int Ny, int planes, bool restr, int tz) {
    const int tx = nod_resid_tx(restr), ty = nod_resid_ty(restr);
    return NodResidGrid{tz, (Nx + tx - 1) / tx, (Ny + ty - 1) / ty, (planes + tz - 1) / tz};
}
// Short chunks while there are too few workgroups to fill the chip, long ones
// where the planes read twice count.  FP64, us: norm of 64^3 nodes 9.0 with 4
// planes / 12.7 with 8, of 128^3 18 with 8 / 20 with 4, of 256^3 94 with 16 /
// 104 with 4; restriction (coarse planes) of 64^3 10.6 with 2 / 15.1 with 4,
// of 128^3 23 with 4 / 25 with 2, of 256^3 122 with 8 / 147 with 2.
template <typename T>
NodResidGrid nod_resid_grid(const NodLevelT<T>& L, int planes, bool restr) {
    const double n = (double)L.nodes();
    const int tz = n < 1e5 ? 1 : (n < 1e6 ? 2 : (n < 4e6 ? 4 : 8));
    return nod_resid_grid_of(L.Nx, L.Ny, planes, restr, restr ? tz : 2 * tz);
}

// C: the coarser level (restricting; any level otherwise).  *nparts: the
// partial rows written.
template <typename T, int kMode>
hipError_t launch_nod_resid(const NodLevelT<T>& L, const NodLevelT<T>& C, double* partials, const NodRefine& ra,
                            int* nparts, hipStream_t st) {
    const bool restr = kMode == kNodRestrict;
    const NodResidGrid g = nod_resid_grid(L, restr ? C.Nz : L.Nz, restr);
    hipLaunchKernelGGL((k_nod_resid<T, kMode>), dim3(g.blocks()), dim3(64, kNodResidWaves), 0, st, L, C, g.tz, g.ntx,
                       g.nty, partials, ra);
    if (nparts) *nparts = g.blocks();
    return hipGetLastError();
}

}  // namespace
}  // namespace mg
