// Run lengths of the batched MLP launches.  Host code only.
//
// A run loads its object's weight fragments once (and the backward merges and
// writes one partial gradient), so long runs are cheaper per tile; but a launch
// covers one MLP shape, and with runs of the tuned length the objects of a shape
// often fill a part of the CUs, or a round and a bit of them.  So the tuned (or
// default) length is the longest one used, and the length is the shortest
// multiple of the quantum that needs no more rounds of `target` blocks than the
// tuned length does.  Measured on gfx950, forward of a step: 16 objects of 18000
// rays together 0.96 -> 0.45 ms, 24 objects of 338571 rays 3.46 -> 3.07; two rounds
// in place of one (512 blocks) 0.56 against 0.51 ms on the 16 objects.  The 128-wide
// FP32 chain runs in the forward's runs (16 objects: backward 2.40 -> 1.96 ms);
// 16-bit backward, 48 objects 10.83 -> 10.64 ms.
#pragma once

#include <cstdint>
#include <vector>

#include "common.h"

namespace prenom {
namespace host {

// Tiles that a block of four waves (forward) or eight (backward) takes at once.  A
// 128-wide FP32 forward has eight waves; half of them idle in runs of four tiles,
// which only a launch of fewer runs than CUs takes.
constexpr int64_t kFwdQuantum = 4, kBwdQuantum = 8;

inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// 16-bit backward blocks that a CU holds at a time.
inline int64_t bwd_blocks_per_cu(const MlpShape& m) { return m.width <= 32 ? 2 : 1; }

// Work items of runs of `run` tiles over objects of `tiles` 16-sample tiles.
inline int64_t run_items(const std::vector<int64_t>& tiles, int64_t run)
{
    int64_t k = 0;
    for (int64_t t : tiles) k += (t + run - 1) / run;
    return k;
}

// Tiles per work item of a launch over them.
inline int64_t run_length(const std::vector<int64_t>& tiles, int64_t most, int64_t quantum, int64_t target)
{
    auto items = [&](int64_t run) { return run_items(tiles, run); };
    const int64_t bound = round_up(items(most), target);
    int64_t lo = 1, hi = round_up(most, quantum) / quantum;  // in quanta; items(hi) <= bound
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (items(mid * quantum) <= bound)
            hi = mid;
        else
            lo = mid + 1;
    }
    return hi * quantum < most ? hi * quantum : most;
}

// Work items that the arrays of such a launch hold: no fewer than run_length
// gives, and no more for fewer tiles (its own number falls where a tile more
// takes a longer run).
inline int64_t run_capacity(const std::vector<int64_t>& tiles, int64_t most, int64_t quantum, int64_t target)
{
    const int64_t a = run_items(tiles, quantum), b = round_up(run_items(tiles, most), target);
    return a < b ? a : b;
}

}  // namespace host
}  // namespace prenom
