// Sizes of launches as plain C++, so that a host compiler can check them.
#pragma once

#include <cstddef>
#include <cstdint>

namespace vqe {

// LDS of a tiled run (k_prun), in bytes from its start.
struct RunLds {
    size_t par;     // (cos, sgn sin) and (sgn, 0) of gate j at par + 32 j
    size_t wsum;    // reverse sweep: wave totals [gates][waves]
    size_t total;
};

// `vectors` (1 forward, 2 reverse) tiles of `entries` amplitudes of vbytes with
// the lists' idle pair each, then the gates.  A pass reads the next gate's
// (cos, sgn sin) during a gate, at the last one too: forward that is one more
// entry after the gates, in reverse the 32 bytes before them (in the tile).
constexpr RunLds tiled_run_lds(int vectors, size_t vbytes, int entries, int gates, int waves) {
    RunLds l{};
    l.par = (size_t(vectors) * size_t(entries + 2) * vbytes + 15) / 16 * 16;
    l.wsum = l.par + 32 * size_t(gates) + 16;
    l.total = l.wsum + (vectors == 2 ? 8 * size_t(gates) * size_t(waves) : 0);
    return l;
}

// States that one launch may hold when each takes `threads` threads of the grid's
// x dimension: HIP takes less than 2^32 of them; a multiple of 8 (states by XCD).
constexpr int states_per_launch(int64_t threads) {
    const int64_t most = int64_t(0xffffffffu) / (threads < 1 ? 1 : threads) / 8 * 8;
    return int(most < 8 ? 8 : most > (1 << 30) ? (1 << 30) : most);
}

}  // namespace vqe
