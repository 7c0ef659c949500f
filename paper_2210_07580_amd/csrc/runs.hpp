// Neighbouring grids as runs (Section 4.2.2, Algorithm 3, Eq. (2)), for
// sparse data in four dimensions and more.
//
// All grids below one level-(D-1) node of the grid tree (a family) share
// their identifier up to the last dimension, so they share the level-(D-1)
// nodes within reach as well; below each such node the grids of Nei(g) are
// one contiguous run of at most 2 w + 1 grids (keys within +-w of g's last
// key), hence also one contiguous run of sorted points.  Sparse data (a few
// points per grid) therefore keeps one list per family (nodes.hip) instead of
// one per grid, and every consumer finds the runs itself while it streams
// the family's list: an entry costs the node's child range and a short key
// search, from arrays that stay in cache, where the written-out lists of a
// 10M-point 5-D call were 20 GB, written once and read two to three times (the
// call: 100 -> 37.5 ms).  In two and three dimensions a list has at most 20 or 116
// entries, a run replaces about three of them, and the searches cost the
// consumers more than the shorter lists save (a batch of 256 instances: lists
// 1.8 -> 0.3 ms, consumers + 2.1 ms): there the lists are kept.
//
// A list entry holds, below the node, how it touches (kSame: equal keys so far;
// kFace, kEdge, kTouch: one, two or more keys differ, each by one; kApart:
// some key differs by more) and the budget d - offset (Eq. (2)) that the next
// levels may still use, which fixes the window w.  The entries that touch come
// first in a list: core marking closes most queries on them, and the merge
// takes them first.  Level-1 nodes need no list: within one instance they are
// in key order, so those within a window of +-3 keys are among the three
// before and the three after.
#pragma once

#include <climits>

#include "common.hpp"
#include "launch.hpp"
#include "walk.hpp"

namespace gd {

constexpr int kSame = 0, kFace = 1, kEdge = 2, kTouch = 3, kApart = 4;
__device__ __forceinline__ uint32_t node_entry(uint32_t node, int touch, int budget) {
    return (node << 6) | ((uint32_t)touch << 3) | (uint32_t)(budget - 1);
}
__device__ __forceinline__ uint32_t entry_node(uint32_t v) { return v >> 6; }
__device__ __forceinline__ int entry_touch(uint32_t v) { return (int)((v >> 3) & 7u); }
__device__ __forceinline__ int entry_budget(uint32_t v) { return (int)(v & 7u) + 1; }
// One more dimension, whose keys differ by ad.
__device__ __forceinline__ int touch_step(int touch, int ad) {
    return touch == kApart || ad > 1 ? kApart : min(touch + ad, kTouch);
}

// Candidate j (0..kNear-1) around a level-1 node: from -first on upwards, then
// the others downwards (first 0: 0, +1, +2, +3, -1, -2, -3; first 3: -3 .. +3).
__device__ __forceinline__ int near_step(int j, int first) { return j - first <= kNear / 2 ? j - first : kNear / 2 - j; }

// Prefix sum within groups of S lanes.
template <int S>
__device__ __forceinline__ uint32_t group_sum_scan(uint32_t v) {
    if constexpr (S == kWave) {
        return wave_incl_scan(v);
    } else if constexpr (S == 16) {
        v += dpp<kRowShr + 1>(0u, v);
        v += dpp<kRowShr + 2>(0u, v);
        v += dpp<kRowShr + 4>(0u, v);
        v += dpp<kRowShr + 8>(0u, v);
        return v;
    } else {
        const int sub = lane_id() % S;
#pragma unroll
        for (int o = 1; o < S; o <<= 1) {
            const uint32_t t = __shfl_up(v, o, S);
            if (sub >= o) v += t;
        }
        return v;
    }
}

// Whether grid c lies behind the first kFamilyGrids of its family f.
__device__ __forceinline__ bool family_rest(const uint32_t* __restrict__ excl, const uint32_t* __restrict__ child,
                                            uint32_t c, uint32_t& f) {
    f = excl[c + 1] - 1;
    return c - child[f] >= kFamilyGrids;
}

struct __attribute__((packed, aligned(4))) Words2 {
    uint32_t v[2];
};
struct __attribute__((packed, aligned(4))) Keys4 {
    int32_t v[4];
};

// Children of node b: [lo, hi), from one 8-byte load.
__device__ __forceinline__ void node_children(const uint32_t* __restrict__ child, uint32_t b, uint32_t& lo,
                                              uint32_t& hi) {
    const Words2 c = *reinterpret_cast<const Words2*>(child + b);
    lo = c.v[0];
    hi = c.v[1];
}

// The children [lo, hi) of a node, among [c0, c1) with ascending keys, whose
// keys lie within +-win (at most 3) of k, and how many of them lie within +-1
// (near).  A binary search leaves at most four places for lo; the keys from
// there on come in 16-byte loads, the later ones only when some lane's node
// goes that far (the work is bound by vector instructions, and most nodes have
// a few children).  Up to three words behind the node's last child may be
// loaded and are not used (every key array is followed by other arrays of the
// workspace, see carve()).  Every lane of the wave's active group calls it.
template <bool kCountNear>
__device__ __forceinline__ void child_window(const int32_t* __restrict__ key, uint32_t c0, uint32_t c1, int32_t k,
                                             int win, uint32_t& lo, uint32_t& hi, uint32_t& near) {
    uint32_t a = c0, b = c1;
    const int32_t want = k - win, last = k + win;
    while (b - a > 4u) {
        const uint32_t m = (a + b) >> 1;
        if (key[m] < want) a = m + 1; else b = m;
    }
    const uint32_t n = c1 - a;  // keys from a on; lo <= a + 4, hi <= lo + 7
    uint32_t below = 0, upto = 0, nb = 0, nu = 0;
#pragma unroll
    for (uint32_t j = 0; j < 12; j += 4) {
        if (j != 0 && !ballot(n > j)) break;
        if (n > j) {
            const Keys4 t = *reinterpret_cast<const Keys4*>(key + a + j);
#pragma unroll
            for (uint32_t v = 0; v < 4; ++v) {
                const int32_t x = j + v < n ? t.v[v] : INT_MAX;
                if (j == 0) below += x < want ? 1u : 0u;
                upto += x <= last ? 1u : 0u;
                if constexpr (kCountNear) {
                    nb += x < k - 1 ? 1u : 0u;
                    nu += x <= k + 1 ? 1u : 0u;
                }
            }
        }
    }
    lo = a + below;
    hi = a + upto;
    near = nu - nb;
}

__device__ __forceinline__ void child_window(const int32_t* __restrict__ key, uint32_t c0, uint32_t c1, int32_t k,
                                             int win, uint32_t& lo, uint32_t& hi) {
    uint32_t near;
    child_window<false>(key, c0, c1, k, win, lo, hi, near);
}

// Grid c's visits: the entries [e0, e1) of its family's list (those below
// e0 + near touch), each giving one run of grids; the own grid is in the run
// of its own family.
template <int D>
struct RunCursor {
    uint64_t e0, e1;
    int32_t k;  // the grid's last key

    __device__ __forceinline__ void open(const RunSource& rs, const GridView& gv, int64_t c) {
        const uint32_t p = rs.excl[c + 1] - 1;
        k = gv.ck[(int64_t)D * gv.ck_stride + c];
        e0 = rs.off[p];
        e1 = rs.off[p + 1];
    }

    // The run of list entry v.
    __device__ __forceinline__ void run_of(const RunSource& rs, uint32_t v, uint32_t& lo, uint32_t& hi) const {
        const int w = walk_window(entry_budget(v));
        uint32_t c0, c1;
        node_children(rs.t.child[D - 1], entry_node(v), c0, c1);
        child_window(rs.t.key[D], c0, c1, k, w, lo, hi);
    }
};

}  // namespace gd
