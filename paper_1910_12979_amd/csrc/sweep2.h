// Two FP32 sweeps of the finest level of a single problem in one launch.
#pragma once

#include "sweep.h"

namespace mg {

// Tile of a workgroup in cells; its march takes six steps more than planes.
constexpr int kPairTX = 56, kPairTY = 24, kPairTZ = 64;

// Whether two sweeps in a row (coefficients from rho, no outflow side) go in
// one launch: where that is the faster way, unless the sweep's tiles are forced
// (tuned ones are for the sweeps that stay single).
// A workgroup fills a compute unit, so the launch costs its rounds of 256
// workgroups times the steps of a chunk, about 1.65 us each; two single sweeps
// cost 3.52 ps a cell each.  256^3 (one round of 220) 111 to 117 us against 118
// to 126, 512^3 (seven) 827 to 875 against 967 to 1088; 288^3 would take two
// rounds, 231 us against 168.
bool sweep_paired(int nx, int ny, int nz);
// in_mode: kInZero, kInPlain or kInProlong, of the first of the two.
hipError_t launch_sweep2(const SweepArgs<float>& a, int in_mode, hipStream_t st);

}  // namespace mg
