// Drives run_ahead (csrc/cycles.h) on a scripted history of residual norms.
//   cycles_ahead FIRST RTOL MAX_CYCLES AHEAD REL_1 REL_2 ...   ("nan": a cycle with a non-finite residual)
// prints: rc status cycles rel over enqueued looks rel_1 rel_2 ...
// The norms go through a ring as on the device: cycle c's in row c mod
// kNormRing, rows that the host has not seen are never overwritten.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "cycles.h"

int main(int argc, char** argv) {
    if (argc < 5) return 2;
    const double first = std::atof(argv[1]), rtol = std::atof(argv[2]), fnorm = 7.0;
    const int max_cycles = std::atoi(argv[3]), width = 4;
    const bool ahead = std::atoi(argv[4]) != 0;
    std::vector<std::string> script(argv + 5, argv + argc);
    std::vector<double> ring(mg::kNormRing * width, -1.0), hist;
    int enqueued = 0, seen = 0, looks = 0;
    auto enqueue = [&](int c) -> int {
        if (c != enqueued || c - seen >= mg::kNormRing || c >= (int)script.size()) return 99;
        const bool bad = script[c] == "nan";
        const double rel = bad ? 1.0 : std::atof(script[c].c_str());
        double* r = ring.data() + c % mg::kNormRing * width;
        r[0] = rel * fnorm * rel * fnorm;
        r[3] = bad ? 1.0 : 0.0;
        ++enqueued;
        return 0;
    };
    auto rows = [&](const double** r) -> int {
        *r = ring.data();
        seen = enqueued;
        ++looks;
        return 0;
    };
    auto record = [&](int c, double rel) {
        if (c == (int)hist.size() + 1) hist.push_back(rel);
    };
    int status = MG_ERR_NOT_CONVERGED, cycles = 0;
    double rel = 1.0;
    bool over = true;
    const int rc = mg::run_ahead(fnorm, rtol, max_cycles, ahead, first, width, &status, &cycles, &rel, &over, enqueue,
                                 rows, record);
    std::printf("%d %d %d %.17g %d %d %d", rc, status, cycles, rel, over ? 1 : 0, enqueued, looks);
    for (double h : hist) std::printf(" %.17g", h);
    std::printf("\n");
    return 0;
}
