// The autotuner's candidates and its search over the binned build's (internal
// header: host code only, checked on the CPU).
#pragma once

#include <cstdint>

namespace dbgrt {

struct Cand {
    bool binned;
    double lf;
    uint32_t block, wpt;
    bool merge;
    uint32_t bin_chunks = 0, bin_div = 0, bin_shape1 = 0, bin_shape2 = 0;
};

// The axes of the search.
constexpr double kLoadFactors[] = {0.5, 0.4, 0.6, 0.7};
constexpr uint32_t kBinChunks[] = {0, 4, 8, 16, 64};  // 0: the default, 32
constexpr uint32_t kBinDivs[] = {0, 1, 2, 4};         // 0: automatic
// scatter shapes, first and second (dbg_config bin_shape1/2): automatic,
// plain tiles, staged lines, big tiles, big tiles then staged lines, wide
// big tiles then big tiles
constexpr uint32_t kBinShapes[][2] = {{0, 0}, {1, 1}, {2, 2}, {3, 3}, {3, 2}, {4, 3}};
constexpr uint32_t kBlocks[] = {256, 512, 1024};
constexpr uint32_t kWpts[] = {2, 4, 8};

// The fastest binned candidate by ms = consider(candidate), 1e300 for one that
// cannot be had: the load factor with automatic shapes, then the scatter shapes
// at the best load factor, then, if set shapes won, the chunks and the second
// scatter's grid divisor.  A build with automatic shapes has neither chunks nor a
// scatter, so with them these would only time one build again and again.
// *best_ms receives its time, *default_ms that of load factor 0.5.
template <typename F>
Cand search_binned(F consider, double *best_ms, double *default_ms) {
    Cand best{true, 0.5, 256, 4, false};
    *best_ms = 1e300;
    const auto attempt = [&](const Cand &c) {
        const double ms = consider(c);
        if (ms < *best_ms) *best_ms = ms, best = c;
        return ms;
    };
    for (double lf : kLoadFactors) {
        const double ms = attempt(Cand{true, lf, 256, 4, false});
        if (lf == 0.5) *default_ms = ms;
    }
    const Cand automatic = best;
    for (const auto &sh : kBinShapes) {
        if (sh[0] == 0 && sh[1] == 0) continue;
        Cand c = automatic;
        c.bin_shape1 = sh[0];
        c.bin_shape2 = sh[1];
        attempt(c);
    }
    if (!best.bin_shape1 && !best.bin_shape2) return best;
    const Cand shaped = best;
    for (uint32_t ch : kBinChunks) {
        if (ch == 0) continue;
        Cand c = shaped;
        c.bin_chunks = ch;
        attempt(c);
    }
    const Cand chunked = best;
    for (uint32_t dv : kBinDivs) {
        if (dv == 0) continue;
        Cand c = chunked;
        c.bin_div = dv;
        attempt(c);
    }
    return best;
}

}  // namespace dbgrt
