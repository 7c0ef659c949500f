// Slots of a queue of tasks that waves reserve side by side (SplitQueue): the
// arithmetic alone, which host programs compile as well.
#pragma once

#include <stdint.h>

namespace gd {

constexpr uint32_t kSplitRows = 2048;  // rows of a task

// Tasks asked for so far.  The counter goes on when the queue is full, so it
// has to hold everything a call may ask for: fewer than 2^31 batches of
// queries (each holds a point), and per batch the slices of neighbours of
// kSplitRows rows and more, at most two per kSplitRows of the call's fewer than
// 2^31 rows, 2^21; less than 2^52 in all.  (32 bits would wrap: 400M points of two
// dimensions in grids of 9e4 with a MinPts of 1e5 ask for 5.5e9, and what comes
// after the wrap would be given slots of others.)
using SplitCount = unsigned long long;

// Whether `want` more tasks fit behind `before` that were asked for earlier.
constexpr bool split_fits(SplitCount before, uint32_t want, uint32_t cap) {
    return before <= cap && want <= cap - before;
}
// Slots in use once `asked` tasks have been asked for.
constexpr uint32_t split_used(SplitCount asked, uint32_t cap) { return asked < cap ? (uint32_t)asked : cap; }

constexpr uint32_t split_slices(uint32_t rows) { return (rows + kSplitRows - 1) / kSplitRows; }

}  // namespace gd
