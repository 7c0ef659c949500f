// Lists of neighbouring tree nodes for sparse data (runs.hpp): for every
// node of level l of the grid tree, the nodes of that level within reach (Eq.
// (2) over the dimensions so far), the node itself included; and, for the last
// level, the lists Nei(g) themselves.
//
// Level by level: the nodes within reach of node a are children of the nodes
// within reach of a's parent, so S lanes per node take the entries of the
// parent's list, find each entry's children within the window (child_window)
// and write them.  All lanes of a group work on one list at every level,
// where a walk per grid from the root (neighbors.hip) is one long chain of
// dependent loads per lane with lanes in different loops.
//
// 10M 5-D points (6.9M grids, 3.1M families): walks counted and wrote 5.1e9
// list entries in 52 ms; these lists hold 0.8e9 and take 9.5 ms.  2M and 1M
// 7-D points: 7.1 -> 0.9 and 5.1 -> 0.6 ms.  The passes over long lists are
// bound by vector instructions (74-91% of the issue rate), most of them the key
// search and the entries' arithmetic; pass 2 therefore writes one entry per
// lane and round rather than each lane its own run (6.3 -> 5.7 ms).  The lists
// of the grids themselves in two and three dimensions: 43 -> 35 us for 20k
// points in two, 131 -> 79 us in three (the read-back between the passes
// included), even at millions of grids; lists by offset of 2M points in seven
// dimensions (5,892 and 10,380 grids) 1,430 -> 250 and 1,456 -> 265 us, in five
// (6,310) 304 -> 145.
#include <algorithm>

#include "launch.hpp"
#include "runs.hpp"
#include "scan.hpp"

namespace gd {

namespace {

struct LevelArgs {
    const Inst* inst;
    const int32_t* key0;        // instance id of each level-0 node
    const uint32_t* child0;
    const uint32_t* par1;       // level-0 node of each level-1 node
    const int32_t* pkey;        // keys of level l - 1 (l == 2: of the level-1 nodes)
    const int32_t* key;         // keys of level l
    const uint32_t* child;      // children of the level-(l-1) nodes
    const uint32_t* par;        // parent of each level-l node
    const uint32_t* excl;       // the last level: level-(D-1) nodes before each grid (par is not kept)
    const uint32_t* nodes;      // device: nodes of level l
    const uint32_t* pnodes;     // device: nodes of level l - 1
    const uint64_t* poff;       // lists of level l - 1 (l >= 3)
    const uint32_t* pent;
    uint64_t pcap;              // entries pent holds
    uint32_t* cnt;              // pass 1: list length of each node
    uint32_t* near;             // touching entries of each node, listed first (nullptr: order kept)
    const uint64_t* off;        // pass 2: where each list goes
    uint32_t* ent;
    uint64_t cap;
    uint2* up;                  // the last level: range of the larger grids in each list, or (kOrdered)
                                // the own grid's place among those at offset 0, and their number
    const int32_t* ck0;         // instance of each grid (count > 1)
    int count;                  // instances
    int first;                  // l == 2: the places around a parent from -first on, then the others
    Header* hdr;
};

// kFirst: l == 2, whose parents' neighbours are the kNear places around them.
// kGrids: l == D, entries are grid indices and the own grid is left out.
// kOrdered (kGrids): lists by offset; the entries are gone through twice, for
// the length of each offset's part and to place them.
template <int S, bool kFirst, bool kGrids, bool kFill, bool kOrdered = false>
__global__ __launch_bounds__(kBlock) void level_kernel(LevelArgs A) {
    constexpr int G = kWave / S;
    // pass 2 of long lists: the chunk's runs, written out one entry per lane
    constexpr bool kFlat = kFill && S == kWave;
    static_assert(!kOrdered || (kFlat && kGrids), "ordered lists are written entry by entry");
    __shared__ uint32_t s_at[kFlat ? kWavesPerBlock : 1][kWave];    // first child of a lane's run, minus its place
    __shared__ uint32_t s_how[kFlat ? kWavesPerBlock : 1][kWave];   // the entry's low bits
    __shared__ uint32_t s_head[kFlat ? kWavesPerBlock : 1][kWave];  // lane + 1 of the run that starts here
    const int lane = lane_id();
    const int sub = lane % S;
    const int64_t nodes = *A.nodes;
    const int64_t a = (xcd_runs<16>(block_id(), block_count()) * kWavesPerBlock + wave_id()) * G + lane / S;
    // a list beyond its buffer (a sync-free run that met more than it was
    // planned for): nothing is read or written
    if (kFill && A.off[nodes] > A.cap) {
        if (block_id() == 0 && threadIdx.x == 0) atomicOr(&A.hdr->err, kErrNeiOverflow);
        return;
    }
    if (!kFirst && A.poff[*A.pnodes] > A.pcap) {
        if (!kFill && a < nodes && sub == 0) A.cnt[a] = 0;
        return;
    }
    if (a >= nodes) return;
    const uint32_t p = kGrids ? A.excl[a + 1] - 1 : A.par[a];
    const int32_t k = A.key[a];
    uint64_t e0 = 0, e1 = kNear, pos = 0;
    uint32_t lo1 = 0, hi1 = 0;
    int32_t k1 = 0;
    int dk = 0;
    if constexpr (kFirst) {
        const uint32_t i0 = A.par1[p];
        lo1 = A.child0[i0];
        hi1 = A.child0[i0 + 1];
        k1 = A.pkey[p];
        dk = A.inst[A.key0[i0]].d;
    } else {
        e0 = A.poff[p];
        e1 = A.poff[p + 1];
    }
    const bool split = !kGrids && A.near != nullptr;
    uint64_t far = 0;  // where the next entry that does not touch goes
    if constexpr (kFill) {
        pos = A.off[a];
        if (split) far = pos + A.near[a];
    }
    uint32_t total = 0, nears = 0;
    uint32_t own = 0, above = 0;  // kGrids: entries before the own grid, entries above it (this lane's)
    const uint64_t pos0 = pos;
    uint32_t part[kMaxD] = {};  // kOrdered: length, then next place, of each offset's part
    uint32_t zeros = 0;         // and the length of the first
    if constexpr (kOrdered) dk = A.inst[A.count == 1 ? 0 : A.ck0[a]].d;
    for (int pass = kOrdered ? 0 : 1; pass < 2; ++pass) {
        for (uint64_t e = e0; e < e1; e += S) {
            if (kOrdered && pass == 1 && e == e0) {
                uint32_t run = 0;
                zeros = part[0];
#pragma unroll
                for (int o = 0; o < kMaxD; ++o) {
                    const uint32_t m = part[o];
                    part[o] = run;
                    run += m;
                }
            }
            bool in = e + sub < e1;
            uint32_t b = 0;
            int budget = 1, touch = 0;
            if constexpr (kFirst) {
                const int64_t x = (int64_t)p + near_step(sub, A.first);
                in = in && x >= (int64_t)lo1 && x < (int64_t)hi1;
                b = in ? (uint32_t)x : p;
                const int dl = A.pkey[b] - k1;
                const int ad = dl < 0 ? -dl : dl;
                in = in && ad <= walk_window(dk);
                const int gap = ad > 0 ? ad - 1 : 0;
                budget = dk - gap * gap;
                touch = touch_step(0, ad);
            } else if (in) {
                const uint32_t v = A.pent[e + sub];
                b = entry_node(v);
                budget = entry_budget(v);
                touch = entry_touch(v);
            }
            uint32_t c0 = 0, c1 = 0, lo, hi, mn;
            if (in) node_children(A.child, b, c0, c1);
            child_window<!kGrids && !kFlat>(A.key, c0, c1, k, walk_window(budget), lo, hi, mn);
            uint32_t m = hi - lo;
            if (!split || touch == kApart) mn = 0;
            if constexpr (!kFill) {
                total += m;
                nears += mn;
            } else if constexpr (kFlat) {
                const int w = wave_id();
                const uint32_t incl = wave_incl_scan(m), excl = incl - m, tot = last_lane(incl);
                s_at[w][lane] = lo - excl;
                s_how[w][lane] = node_entry(0u, touch, budget);
                uint32_t carry = 0;
                for (uint32_t t0 = 0; t0 < tot; t0 += kWave) {
                    // the run of each place: see core_mark_runs_kernel
                    s_head[w][lane] = 0;
                    wave_sync();
                    if (m != 0 && excl >= t0 && excl < t0 + kWave) s_head[w][excl - t0] = (uint32_t)lane + 1u;
                    wave_sync();
                    uint32_t j = wave_max_scan(s_head[w][lane]);
                    j = j ? j : carry;
                    carry = last_lane(j);
                    j = (j ? j : 1u) - 1u;
                    bool v = t0 + lane < tot;
                    const uint32_t x = v ? s_at[w][j] + t0 + lane : (uint32_t)a;
                    const uint64_t lt = lanemask_lt();
                    if constexpr (kGrids && !kOrdered) {
                        const uint64_t sm = ballot(v && x == (uint32_t)a);
                        v = v && x != (uint32_t)a;
                        const uint64_t vm = ballot(v);
                        if (v) A.ent[pos + popc64(vm & lt)] = x;
                        above += v && x > (uint32_t)a ? 1u : 0u;
                        if (sm && lane == 0) own = (uint32_t)(pos - pos0) + (uint32_t)popc64(vm & ((sm & -sm) - 1ull));
                        pos += popc64(vm);
                        continue;
                    }
                    const uint32_t how = s_how[w][j];
                    const int dl = A.key[x] - k;
                    const int ad = dl < 0 ? -dl : dl;
                    const int gap = ad > 0 ? ad - 1 : 0;
                    const int left = entry_budget(how) - gap * gap;
                    if constexpr (kOrdered) {
                        const bool self = v && x == (uint32_t)a;
                        const int off = v && !self ? dk - left : kMaxD;
                        const uint64_t sm = ballot(self);
                        if (pass == 1 && sm) own = part[0] + (uint32_t)popc64(ballot(off == 0) & ((sm & -sm) - 1ull));
                        uint32_t at = 0;
#pragma unroll
                        for (int o = 0; o < kMaxD; ++o) {
                            if (o >= dk) continue;
                            const uint64_t om = ballot(off == o);
                            if (off == o) at = part[o] + (uint32_t)popc64(om & lt);
                            part[o] += (uint32_t)popc64(om);
                        }
                        if (pass == 1 && off != kMaxD) A.ent[pos0 + at] = x;
                        continue;
                    }
                    const int t = touch_step(entry_touch(how), ad);
                    const uint32_t y = node_entry(x, t, left);
                    const uint64_t nm = ballot(v && split && t != kApart), fm = ballot(v) & ~nm;
                    const bool nr = (nm >> lane) & 1ull;
                    uint64_t& fpos = split ? far : pos;
                    const uint64_t to = nr ? pos + popc64(nm & lt) : fpos + popc64(fm & lt);
                    if (v) A.ent[to] = y;
                    fpos += popc64(fm);
                    if (split) pos += popc64(nm);
                }
                wave_sync();
            } else {
                // the own grid is written nowhere
                if (kGrids && in && b == p) --m;
                const uint32_t f = m - mn;
                const uint32_t fi = group_sum_scan<S>(f), ni = split ? group_sum_scan<S>(mn) : 0u;
                uint64_t wf = (split ? far : pos) + (fi - f), wn = pos + (ni - mn);
                for (uint32_t x = lo; x < hi; ++x) {
                    if constexpr (kGrids) {
                        if (x == (uint32_t)a) {
                            own = (uint32_t)(wf - pos0);
                        } else {
                            A.ent[wf++] = x;
                            above += x > (uint32_t)a ? 1u : 0u;
                        }
                    } else {
                        const int dl = A.key[x] - k;
                        const int ad = dl < 0 ? -dl : dl;
                        const int gap = ad > 0 ? ad - 1 : 0;
                        const int t = touch_step(touch, ad);
                        uint64_t& to = split && t != kApart ? wn : wf;
                        A.ent[to++] = node_entry(x, t, budget - gap * gap);
                    }
                }
                const uint32_t ft = __shfl(fi, S - 1, S);
                if (split) {
                    far += ft;
                    pos += __shfl(ni, S - 1, S);
                } else {
                    pos += ft;
                }
            }
        }
    }
    if constexpr (!kFill) {
#pragma unroll
        for (int o = S / 2; o > 0; o >>= 1) {
            total += __shfl_xor(total, o, S);
            nears += __shfl_xor(nears, o, S);
        }
        if (sub == 0) {
            A.cnt[a] = total - (kGrids ? 1u : 0u);
            if (split) A.near[a] = nears;
        }
    } else if constexpr (kOrdered) {
        if (lane == 0) A.up[a] = make_uint2(own, zeros);
    } else if constexpr (kGrids) {
#pragma unroll
        for (int o = S / 2; o > 0; o >>= 1) {
            own += __shfl_xor(own, o, S);
            above += __shfl_xor(above, o, S);
        }
        if (sub == 0) A.up[a] = make_uint2(own, own + above);
    }
}

// Neighbours of all grids (their own included), counted in the runs: a wave takes
// kCountFamilies families one after another (in the waves behind: 64 grids that
// lie behind the first kFamilyGrids of theirs), a lane the entry, whose window is
// searched for each of the family's grids.  Entries (p, b) and (b, p) count the
// same pairs: those with b > p count twice.  A walk of the tree per grid takes
// 18.8 ms where this takes 14.2 (10M 5-D points, 5.1e9 neighbours), 3.2 and 0.2
// (2M 7-D).
constexpr int kCountFamilies = 8;

__global__ __launch_bounds__(kBlock) void run_total_kernel(const uint32_t* families, const uint32_t* ncell,
                                                           RunSource rs, const uint32_t* __restrict__ child,
                                                           const int32_t* __restrict__ key, int64_t family_waves,
                                                           uint64_t* total) {
    __shared__ uint64_t sums[kWavesPerBlock];
    const int w = wave_id(), lane = lane_id();
    const int64_t wave = xcd_runs<16>(block_id(), block_count()) * kWavesPerBlock + w;
    uint64_t sum = 0;
    auto count = [&](uint32_t p, uint32_t cb, uint32_t m) {  // grids [cb, cb + m) of family p, m at most 64
        const int32_t keys = key[cb + min((uint32_t)lane, m - 1)];
        const uint64_t e1 = rs.off[p + 1];
        for (uint64_t e = rs.off[p]; e < e1; e += kWave) {
            const uint32_t v = e + lane < e1 ? rs.ent[e + lane] : 0u;
            const uint32_t b = entry_node(v);
            const bool in = e + lane < e1 && b >= p;
            if (!ballot(in)) continue;
            uint32_t b0 = 0, b1 = 0, pairs = 0;
            if (in) node_children(child, b, b0, b1);
            for (uint32_t a = 0; a < m; ++a) {
                uint32_t lo, hi;
                child_window(key, b0, b1, readlane(keys, (int)a), walk_window(entry_budget(v)), lo, hi);
                pairs += hi - lo;
            }
            sum += b == p ? (uint64_t)pairs : 2ull * pairs;
        }
    };
    if (wave < family_waves) {
        const int64_t f0 = wave * kCountFamilies, f1 = min(f0 + kCountFamilies, (int64_t)*families);
        for (int64_t f = f0; f < f1; ++f) {
            const uint32_t c0 = child[f];
            count((uint32_t)f, c0, min(child[f + 1] - c0, kFamilyGrids));
        }
    } else {
        const int64_t c = (wave - family_waves) * kWave + lane;
        uint32_t f = 0;
        const bool mine = c < (int64_t)*ncell && family_rest(rs.excl, child, (uint32_t)c, f);
        for (uint64_t todo = ballot(mine); todo;) {
            const int first = ffs64(todo);
            const uint32_t p = readlane(f, first);
            const uint64_t same = ballot(mine && f == p);
            todo &= ~same;
            count(p, (uint32_t)(c - lane) + (uint32_t)first, (uint32_t)popc64(same));
        }
    }
    sum = wave_sum(sum);
    if (lane == 0) sums[w] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kWavesPerBlock; ++i) sum += sums[i];
        if (sum) atomicAdd((unsigned long long*)total, (unsigned long long)sum);
    }
}

struct NodeTotal {
    const uint32_t* cnt;
    const uint32_t* nodes;
    __device__ uint64_t operator()(int64_t a) const { return a < (int64_t)*nodes ? (uint64_t)cnt[a] : 0ull; }
};

struct NodeOffWriter {
    uint64_t* off;
    const uint32_t* nodes;
    uint64_t* total;
    __device__ void operator()(int64_t a, uint64_t ex, uint64_t) const {
        if (a > (int64_t)*nodes) return;
        off[a] = ex;
        if (a == (int64_t)*nodes) *total = ex;
    }
};

LevelArgs level_args(const GridView& g, const TreeView& t, const NodeLists& nl, int l) {
    LevelArgs A{};
    A.inst = g.b.inst;
    A.key0 = t.key[0];
    A.child0 = t.child[0];
    A.par1 = nl.par[1];
    A.pkey = t.key[l - 1];
    A.key = t.key[l];
    A.child = t.child[l - 1];
    A.par = nl.par[l];
    A.excl = nl.excl;
    A.nodes = t.level_count + l;
    A.pnodes = t.level_count + (l - 1);
    A.poff = nl.off[(l - 1) & 1];
    A.pent = nl.ent[(l - 1) & 1];
    A.pcap = nl.cap[(l - 1) & 1];
    A.cnt = nl.cnt;
    A.near = nl.near;
    A.off = nl.off[l & 1];
    A.ent = nl.ent[l & 1];
    A.cap = nl.cap[l & 1];
    A.up = nl.up;
    A.ck0 = g.ck;
    A.count = g.b.count;
    A.first = nl.ordered ? kNear / 2 : 0;
    A.hdr = g.b.hdr;
    return A;
}

template <bool kFill>
hipError_t launch_level(const GridView& g, const LevelArgs& A, int l, int64_t nodes, int lanes, bool ordered,
                        hipStream_t st) {
    const dim3 threads(kBlock);
    auto blocks = [&](int S) { return grid_of((nodes * S + kBlock - 1) / kBlock); };
    const bool grids = l == g.D;
    if (l == 2 && grids)
        level_kernel<8, true, true, kFill><<<blocks(8), threads, 0, st>>>(A);
    else if (l == 2)
        level_kernel<8, true, false, kFill><<<blocks(8), threads, 0, st>>>(A);
    else if (grids && lanes == 8)
        level_kernel<8, false, true, kFill><<<blocks(8), threads, 0, st>>>(A);
    else if (grids && lanes == 16)
        level_kernel<16, false, true, kFill><<<blocks(16), threads, 0, st>>>(A);
    else if (grids && ordered && kFill)
        level_kernel<kWave, false, true, kFill, kFill><<<blocks(kWave), threads, 0, st>>>(A);
    else if (grids)
        level_kernel<kWave, false, true, kFill><<<blocks(kWave), threads, 0, st>>>(A);
    else if (lanes <= 16)
        level_kernel<16, false, false, kFill><<<blocks(16), threads, 0, st>>>(A);
    else
        level_kernel<kWave, false, false, kFill><<<blocks(kWave), threads, 0, st>>>(A);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_run_total(const GridView& g, const RunSource& runs, hipStream_t st) {
    if (g.ncell == 0) return hipSuccess;
    const int64_t per_block = (int64_t)kWavesPerBlock * kCountFamilies;
    const int64_t blocks = (runs.families + per_block - 1) / per_block;
    const int64_t rest = runs.long_families ? grid_for(g.ncell, kWavesPerBlock * kWave) : 0;
    run_total_kernel<<<grid_of(blocks + rest), dim3(kBlock), 0, st>>>(
        runs.t.level_count + (g.D - 1), g.ncell_dev, runs, runs.t.child[g.D - 1], runs.t.key[g.D],
        blocks * kWavesPerBlock, &g.b.hdr->run_total);
    return hipGetLastError();
}

hipError_t launch_level_count(const GridView& g, const TreeView& t, const NodeLists& nl, int l, int64_t nodes,
                              int lanes, uint64_t* partial, hipStream_t st) {
    if (nodes <= 0) return hipSuccess;
    const LevelArgs A = level_args(g, t, nl, l);
    const hipError_t e = launch_level<false>(g, A, l, nodes, lanes, nl.ordered, st);
    if (e != hipSuccess) return e;
    return scan_apply<uint64_t>(NodeTotal{nl.cnt, A.nodes}, nodes + 1,
                                NodeOffWriter{nl.off[l & 1], A.nodes, &g.b.hdr->nei_total}, (uint64_t*)nullptr, partial,
                                st);
}

hipError_t launch_level_fill(const GridView& g, const TreeView& t, const NodeLists& nl, int l, int64_t nodes,
                             int lanes, hipStream_t st) {
    if (nodes <= 0) return hipSuccess;
    return launch_level<true>(g, level_args(g, t, nl, l), l, nodes, lanes, nl.ordered, st);
}

}  // namespace gd
