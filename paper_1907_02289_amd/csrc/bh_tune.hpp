// bh_tune.hpp -- the choice that bh_autotune makes from its measured times:
// host arithmetic only.
#pragma once

namespace bhk {

// Times (ms) of one group size: the force kernel with tiles of 512 and 256
// sources, and the walk.
struct TuneTimes {
    double force512, force256, walk;
};

// A group size's tile, by its force times alone: 256 wins by 2% or not at all,
// as single timings differ by that much.
inline int tune_tile(const TuneTimes &t) { return t.force256 * 1.02 < t.force512 ? 256 : 512; }

// A group size's time per step with that tile and lists kept for rebuild_every evaluations.
inline double tune_cost(const TuneTimes &t, int tile, int rebuild_every) {
    return (tile == 256 ? t.force256 : t.force512) + t.walk / rebuild_every;
}

}  // namespace bhk
