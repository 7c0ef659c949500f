// Capacities of a planned (captured) run from what the eager call before it
// met: a sixteenth and a little more, within what the kernels can hold.  The
// arithmetic alone, which host programs compile as well.
#pragma once

#include <stdint.h>

namespace gd {

// Node lists and runs hold a node above the 6 bits of its entry (runs.hpp), in 32
// bits: a call with this many grids, or a plan for as many, does without them.
constexpr int64_t kMaxRunNodes = (int64_t)1 << 26;

constexpr int64_t at_most(int64_t v, int64_t bound) { return v < bound ? v : bound; }

// Grids of a call of n points.  levels: its lists are built level by level or
// read as runs, and a replay with more nodes than an entry can name has to be
// refused by the grid count.
constexpr int64_t planned_grids(int64_t n, int64_t grids, bool levels) {
    const int64_t most = at_most(n, grids + grids / 16 + 1024);
    return levels ? at_most(most, kMaxRunNodes - 1) : most;
}
// Nodes of one tree level of a call planned for ncell grids.
constexpr int64_t planned_nodes(int64_t ncell, int64_t nodes) { return at_most(ncell, nodes + nodes / 16 + 1024); }

}  // namespace gd
