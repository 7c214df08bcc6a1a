// The iterations of a solve, enqueued ahead of their residual norms.  Host
// code only: what enqueues a cycle and what reads the norms are the caller's.
#pragma once

#include <algorithm>
#include <cmath>

#include "../../include/macproj.h"

namespace mg {

// Residual norms kept on the device, the c-th cycle's (from 0) in row c mod
// kNormRing, so that several cycles can run before the host looks.
constexpr int kNormRing = 8;

// The ratio of successive residual norms below which the first cycle of a
// solve tells how the next ones will go, per V-cycle it runs (norm_ahead).
constexpr double kFirstGainMac = 0.02;
constexpr double kFirstGainNodal = 0.01;

// How many cycles to enqueue before looking at the next residual norm: as many
// as are sure to be needed (rel: the last relative residual, known: the ratios
// of successive ones seen so far, best: the smallest of them, room: cycles
// allowed).  A cycle counts as needed if the residual ahead of it, at ten
// times below what the best ratio predicts, is above rtol.
// From the second cycle on the ratio is nearly constant and slowly worsens.
// The first one depends on the right-hand side: random velocities leave 0.008
// (then 0.03, 0.04, ..), but a smooth f leaves 0.2 to 0.9 of its residual and
// then 0.02, 0.04, so that the first ratio alone sent a third of such solves
// past their convergence, to be run again (128^3, rtol 1e-6: 3.16 ms, now
// 1.40).  It is trusted only at or below `first`; else the second is waited
// for.  Of 504 smooth and rough f at 92 tolerances none is run again then.
inline int norm_ahead(double rel, double best, int known, double first, double rtol, int room) {
    int m = 1;
    if (known == 0 || (known == 1 && best > first) || !(best > 0.0 && best < 1.0)) return m;
    for (double p = rel * best; m < kNormRing && m < room && p > 10.0 * rtol; p *= best) ++m;
    return m;
}

// enqueue(c) puts cycle c (from 0) on its stream; rows(&r) waits for them and
// gives the ring's rows {||r||^2, -, -, #non-finite}, `width` doubles each;
// record(c, rel) takes the history.  *status, *cycles and *rel are the
// caller's start values and the solve's results.  ahead: look ahead as
// norm_ahead allows.  *over: converged before the last cycle enqueued, so that
// the solve has to be run again without looking ahead.
template <typename E, typename R, typename Rec>
int run_ahead(double fnorm, double rtol, int max_cycles, bool ahead, double first, int width, int* status, int* cycles,
              double* rel, bool* over, E&& enqueue, R&& rows, Rec&& record) {
    double best = 0.0;
    int known = 0;
    *over = false;
    while (*status == MG_ERR_NOT_CONVERGED && *cycles < max_cycles) {
        const int m = ahead ? norm_ahead(*rel, best, known, first, rtol, max_cycles - *cycles) : 1;
        for (int i = 0; i < m; ++i) {
            int rc = enqueue(*cycles + i);
            if (rc) return rc;
        }
        const double* ring = nullptr;
        int rc = rows(&ring);
        if (rc) return rc;
        for (int i = 0; i < m; ++i) {
            const double* r = ring + *cycles % kNormRing * width;
            const double was = *rel;
            *rel = std::sqrt(r[0]) / fnorm;
            ++*cycles;
            record(*cycles, *rel);
            if (r[3] > 0.0 || !std::isfinite(*rel)) {
                *status = MG_ERR_NONFINITE;
                return MG_OK;
            }
            if (*rel <= rtol) {
                *status = MG_OK;
                *over = i + 1 < m;
                return MG_OK;
            }
            best = known == 0 ? *rel / was : std::min(best, *rel / was);
            ++known;
        }
    }
    return MG_OK;
}

}  // namespace mg
