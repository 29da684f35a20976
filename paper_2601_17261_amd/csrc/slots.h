// On how many workgroups per XCD a forward runs beside other work.  (Host only)
#pragma once
#include <stdint.h>

namespace agzo {

// One problem of 8 x run tiles, tile_us each, in a launch of its own whose workgroups take whole rounds of tiles together, beside a chain of launches
// that takes latency_us + sweep_us by itself, of which only the second depends on how many compute units it has (29 GB/s each, of the 22 that
// each has of the rate of all together), and that goes on with all of them behind the forward; against both one after the other, fork_us
// (a fork and a join) less.  slots: compute units of an XCD.  The workgroups per XCD for which both are done first, 0: one after the
// other; four compute units of each XCD at least are left, so 0 where there are no more than these
inline int lone_slots(int64_t run, int slots, double tile_us, double latency_us, double sweep_us, double fork_us) {
    if (slots <= 4) return 0;
    const double all = latency_us + sweep_us;
    auto rounds = [&](int s) { return (double)((run + s - 1) / s) * tile_us; };
    int best = 0;
    double best_us = rounds(slots) + all - fork_us;
    for (int s = slots - 4; s >= 1; --s) {
        const double left = 22.0 / 29.0 * slots / (slots - s), slow = latency_us + sweep_us * (left > 1.0 ? left : 1.0);
        const double done = rounds(s) / slow, us = done >= 1.0 ? rounds(s) : rounds(s) + (1.0 - done) * all;
        if (us <= best_us) { best_us = us; best = s; }      // (of equal ones the fewest)
    }
    return best;
}

}  // namespace agzo
