// Core points (Definition 1; identified "like G13", Section 3.2 and Section
// 4.4 step 2) and the per-grid core sets s_i used by the merge (Section
// 4.3.1), plus the low-density-first order of the LDF variant (Section 5.2).
//
// A core set is a run of point rows (see CoreOut): a grid whose points are
// all core uses its sorted rows as they are, so only grids that mix core and
// non-core points copy anything.
//
// Marking runs one wave per grid (core_mark_group_kernel: four grids per wave
// where grids and lists are small; core_mark_runs_kernel: neighbours as runs;
// core_tasks_kernel: long streams of few large grids split up).  A grid with at least MinPts points is all
// core (its diameter is below eps).  In a sparser grid every point already
// has the grid's own points as neighbours; the wave then streams the points
// of Nei(g), nearest grids first, as one flat list: each lane owns one
// neighbour grid of a 64-grid chunk, a wave prefix sum of their sizes maps
// every flat item to its grid (binary search over 64 LDS entries), and each
// lane loads one candidate point per step.  The grid's own points are the
// queries: for each still-open query the wave evaluates 64 candidates at
// once, counts the hits with one ballot + popcount, and closes the query as
// soon as its count reaches MinPts (early exit).
#include "launch.hpp"
#include "radix.hpp"
#include "runs.hpp"

namespace gd {

// Squared distance of two points of neighbouring grids: every coordinate
// difference is below 2.13 eps < 2^16 in magnitude, so each square is an
// exact unsigned 24-bit product, and the sum (below 9 eps^2 < 2^32 for
// eps <= 21845) is exact in unsigned 32-bit arithmetic.
// Above that bound (the wide path) the sum is taken in 64 bits.
template <int D, bool kWide>
__device__ __forceinline__ typename Dist<kWide>::T sqdist_nb(const int32_t (&a)[D], const int32_t (&b)[D]) {
    typename Dist<kWide>::T dd = 0;
#pragma unroll
    for (int j = 0; j < D; ++j) dd += sqd<kWide>(a[j], b[j]);
    return dd;
}

// Packed form for small eps: points of neighbouring grids differ by less
// than (2 + sqrt(d - 1)) eps / sqrt(d) <= 2.13 eps per coordinate (the key
// offsets of Eq. (2) bound |k_j - k'_j| by 1 + sqrt(d - 1)), so for
// eps <= kPackedEpsMax every difference fits a signed 16-bit half and the
// squared distance (at most d (2.13 eps)^2 < 2^31) is exact in 32 bits.  Two
// coordinates share a word (low 16 bits of each; a 16-bit difference of the
// low halves is the exact difference when that is below 2^15), one packed
// subtraction and one two-term dot product handle both; an odd last
// coordinate stays a full word.

typedef short short2_t __attribute__((ext_vector_type(2)));

template <int D>
constexpr int packed_words() { return (D + 1) / 2; }

template <int D>
__device__ __forceinline__ void pack_row(const int32_t (&x)[D], int32_t (&p)[packed_words<D>()]) {
#pragma unroll
    for (int w = 0; w < D / 2; ++w) p[w] = (int32_t)(((uint32_t)x[2 * w] & 0xFFFFu) | ((uint32_t)x[2 * w + 1] << 16));
    if constexpr (D & 1) p[D / 2] = x[D - 1];
}

template <int D>
__device__ __forceinline__ uint32_t sqdist_pk(const int32_t (&a)[packed_words<D>()],
                                              const int32_t (&b)[packed_words<D>()]) {
    int32_t acc = 0;
#pragma unroll
    for (int w = 0; w < D / 2; ++w) {
        const short2_t t = __builtin_bit_cast(short2_t, a[w]) - __builtin_bit_cast(short2_t, b[w]);
        acc = __builtin_amdgcn_sdot2(t, t, acc, false);
    }
    if constexpr (D & 1) {
        const int32_t t = a[D / 2] - b[D / 2];
        acc = __mul24(t, t) + acc;
    }
    return (uint32_t)acc;
}

// Candidates of one list step above which a grid leaves its group of 16 lanes.
constexpr uint32_t kGroupStream = 256;

// R: candidate rows per lane per step.  The slowest grids stream dozens of
// steps one after another, each a chain of dependent rounds, so with a large
// MinPts (a query needs more hits than one 64-candidate step can give) a
// step takes two rows; with a small MinPts most queries close within the
// first 64 candidates and a second row would only add distance tests.
template <int D, bool kStats, bool kPacked, int R, bool kWide, bool kSplit>
__global__ __launch_bounds__(kBlock) void core_mark_kernel(GridView gv, const uint64_t* __restrict__ nei_off,
                                                           const uint32_t* __restrict__ nei,
                                                           const uint2* __restrict__ mid, uint8_t* __restrict__ core,
                                                           uint32_t* __restrict__ core_cnt, CoreStats* stats,
                                                           SplitQueue sq) {
    constexpr int PW = packed_words<D>();
    constexpr int S = row_stride(D);
    __shared__ uint32_t s_row[kWavesPerBlock][kWave];   // first row of each lane's grid, minus its place
    __shared__ uint32_t s_head[kWavesPerBlock][kWave];  // its place, or (R = 2) lane + 1 of the grid that starts at this candidate
    __shared__ __align__(16) int32_t s_q[kWavesPerBlock][kWave * S];  // the query rows of the batch
    const int w = wave_id(), lane = lane_id();
    const int64_t c = xcd_runs<16>(block_id(), block_count()) * kWavesPerBlock + w;
    if (c >= (int64_t)*gv.ncell_dev) return;
    // every load that depends on c alone is issued before the first use
    const Inst& I = cell_inst(gv, c);
    const uint32_t st = gv.cell_start[c];
    const uint32_t en = gv.cell_start[c + 1];
    const uint64_t e0 = nei_off[c], e1 = nei_off[c + 1];
    const uint32_t minpts = (uint32_t)I.minpts;
    const typename Dist<kWide>::T T = inst_T<kWide>(I);
    const uint32_t k = en - st;
    if (kPacked && I.eps > kPackedEpsMax) {
        // a replayed graph met a larger eps than it was captured for: the
        // packed differences could wrap, so the run is discarded
        if (lane == 0) atomicOr(&gv.b.hdr->err, kErrPlan);
        return;
    }
    if (k >= minpts) {
        for (uint32_t i = lane; i < k; i += kWave) core[st + i] = 1;
        if (lane == 0) core_cnt[c] = k;
        return;
    }
    const uint32_t need = minpts - k;
    // The neighbours at offset 0 lead the list in ascending order; the 64
    // around the grid's own place among them are the nearest in the first
    // dimensions, so the stream starts there and takes the rest of the
    // offset after (7-D lists of hundreds of entries: 160 -> 67 us; the merge
    // wants the ascending order, 1.3 against 2.9 ms with the nearest first).
    uint32_t first = 0, zeros = 0;
    if (mid) {
        const uint2 m = mid[c];
        zeros = m.y;
        first = m.x > kWave / 2 ? m.x - kWave / 2 : 0u;
    }
    unsigned long long ndist = 0, npts = 0, ncells = 0;
    uint32_t m = 0, tasks = 0;
    for (uint32_t qb = 0; qb < k; qb += kWave) {
        const uint32_t nq = min((uint32_t)kWave, k - qb);
        uint64_t active = nq == (uint32_t)kWave ? ~0ull : ((1ull << nq) - 1ull);
        {
            int32_t qx[D];
            load_row<D>(gv.crd, (uint32_t)lane < nq ? st + qb + lane : st, qx);
            if constexpr (kPacked) {
                int32_t pq[PW];
                pack_row<D>(qx, pq);
                store_row<PW>(s_q[w], lane, pq);
            } else {
                store_row<D>(s_q[w], lane, qx);
            }
        }
        uint32_t mycnt = 0;  // lane i: hits of query i
        // kSplit: neighbours of kSplitRows points and more wait for the second
        // pass, which hands them out as tasks (or streams them if the queue
        // is full)
        bool later = false;
        auto stream = [&](bool large) {
            for (uint64_t e = e0; e < e1 && active; e += kWave) {
                const uint64_t idx = e + lane;
                const bool v = idx < e1;
                uint64_t at = idx;
                if (idx - e0 < zeros) at = idx - e0 + first < zeros ? idx + first : idx + first - zeros;
                const uint32_t cc = v ? nei[at] : 0u;
                const uint32_t cs = v ? gv.cell_start[cc] : 0u;
                uint32_t cn = v ? gv.cell_start[cc + 1] - cs : 0u;
                if constexpr (kSplit) {
                    if ((cn >= kSplitRows) != large) {
                        later |= cn >= kSplitRows;
                        cn = 0;
                    }
                }
                const uint32_t incl = wave_incl_scan(cn);
                const uint32_t tot = last_lane(incl);
                const uint32_t excl = incl - cn;
                s_row[w][lane] = cs - excl;
                if constexpr (R == 1) {
                    s_head[w][lane] = excl;
                    wave_sync();
                }
                // Row of flat candidate t0 + lane.  Long streams (R = 2): the
                // grids that start within the step mark their first candidate,
                // a running maximum over the lanes gives each candidate its
                // grid, and the last one carries over to the next step (10M
                // 3-D points 98 -> 93 us).  Short ones: a binary search over the
                // chunk's 64 grids (the batch of 256 2.21 against 2.29 ms).
                uint32_t carry = 0;
                auto cand_row = [&](uint32_t t0) -> uint32_t {
                    if constexpr (R == 1) {
                        int j = 0;
#pragma unroll
                        for (int step = 32; step > 0; step >>= 1)
                            if (s_head[w][j + step] <= t0 + lane) j += step;
                        return s_row[w][j] + t0 + lane;
                    }
                    s_head[w][lane] = 0;
                    wave_sync();
                    if (cn != 0 && excl >= t0 && excl < t0 + kWave) s_head[w][excl - t0] = (uint32_t)lane + 1u;
                    wave_sync();
                    uint32_t own = wave_max_scan(s_head[w][lane]);
                    own = own ? own : carry;
                    carry = last_lane(own);
                    return s_row[w][(own ? own : 1u) - 1u] + t0 + lane;
                };
                // R candidates per lane per step (64 R per step), and the next
                // step's candidates load while this one is evaluated
                int32_t y[R][D];
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    uint32_t r = st;
                    if ((uint32_t)(u * kWave) < tot) r = cand_row((uint32_t)(u * kWave));
                    load_row<D>(gv.crd, (uint32_t)(u * kWave + lane) < tot ? r : st, y[u]);
                }
                for (uint32_t t0 = 0; t0 < tot && active; t0 += R * kWave) {
                    uint64_t tvm[R];
#pragma unroll
                    for (int u = 0; u < R; ++u) tvm[u] = ballot(t0 + u * kWave + lane < tot);
                    int32_t yn[R][D];
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        const uint32_t tn = t0 + (R + u) * kWave;
                        uint32_t r = st;
                        if (tn < tot) r = cand_row(tn);
                        load_row<D>(gv.crd, tn + lane < tot ? r : st, yn[u]);
                    }
                    int32_t yp[R][PW];
                    if constexpr (kPacked) {
#pragma unroll
                        for (int u = 0; u < R; ++u) pack_row<D>(y[u], yp[u]);
                    }
                    // every open query against the step's candidates, two queries
                    // per round so their LDS reads overlap: the query row comes
                    // from LDS (one broadcast read), lane qi keeps query qi's
                    // hits; counts and closings are folded in once per step
                    const uint64_t act0 = uniform64(active);
                    uint32_t step_hits = 0;
                    for (uint64_t act = act0; act;) {
                        const int qa = ffs64(act);
                        act &= act - 1ull;
                        const int qb2 = act ? ffs64(act) : qa;
                        act &= act - 1ull;
                        uint32_t ha = 0, hb = 0;
                        if constexpr (kPacked) {
                            int32_t pa[PW], pb[PW];
                            load_row<PW>(s_q[w], qa, pa);
                            load_row<PW>(s_q[w], qb2, pb);
#pragma unroll
                            for (int u = 0; u < R; ++u) {
                                ha += (uint32_t)popc64(ballot(sqdist_pk<D>(yp[u], pa) <= T) & tvm[u]);
                                hb += (uint32_t)popc64(ballot(sqdist_pk<D>(yp[u], pb) <= T) & tvm[u]);
                            }
                        } else {
                            int32_t pa[D], pb[D];
                            load_row<D>(s_q[w], qa, pa);
                            load_row<D>(s_q[w], qb2, pb);
#pragma unroll
                            for (int u = 0; u < R; ++u) {
                                ha += (uint32_t)popc64(ballot(sqdist_nb<D, kWide>(y[u], pa) <= T) & tvm[u]);
                                hb += (uint32_t)popc64(ballot(sqdist_nb<D, kWide>(y[u], pb) <= T) & tvm[u]);
                            }
                        }
                        step_hits = lane == qa ? ha : step_hits;
                        step_hits = lane == qb2 ? hb : step_hits;
                        if constexpr (kStats) ndist += (qb2 != qa ? 2u : 1u) * min(tot - t0, (uint32_t)(R * kWave));
                    }
                    mycnt += step_hits;
                    active = act0 & ~ballot(((act0 >> lane) & 1ull) && mycnt >= need);
                    if constexpr (kStats) npts += min(tot - t0, (uint32_t)(R * kWave));
#pragma unroll
                    for (int u = 0; u < R; ++u)
#pragma unroll
                        for (int j = 0; j < D; ++j) y[u][j] = yn[u][j];
                }
                if constexpr (kStats) ncells += large ? 0ull : (unsigned long long)min(e1 - e, (uint64_t)kWave);
                wave_sync();
            }
        };
        stream(false);
        if constexpr (kSplit) {
            if (active && ballot(later)) {
                // the noise points of a sparse grid stream every neighbour, but a
                // large grid counts only if an open query comes within eps of
                // its cell; the rows are read again here, since kept through
                // the stream they cost it registers
                const double side = (double)I.eps / sqrt((double)I.d);
                const double lim = (double)I.eps * (double)I.eps * (1.0 + 1e-9) + 1.0;
                int32_t qx[D];
                load_row<D>(gv.crd, (uint32_t)lane < nq ? st + qb + lane : st, qx);
                auto slices = [&](uint64_t idx, uint32_t& cc) -> uint32_t {
                    cc = idx < e1 ? nei[idx] : 0u;
                    const uint32_t cn = idx < e1 ? gv.cell_start[cc + 1] - gv.cell_start[cc] : 0u;
                    bool take = cn >= kSplitRows;
                    if constexpr (D <= 4) take = take && cell_near<D>(gv, cc, active, qx, side, lim);
                    return take ? split_slices(cn) : 0u;
                };
                uint32_t total = 0, base, cc;
                for (uint64_t e = e0; e < e1; e += kWave) total += wave_sum(slices(e + lane, cc));
                if (total != 0 && split_reserve(sq, total, base)) {
                    tasks += total;
                    for (uint64_t e = e0; e < e1; e += kWave) {
                        const uint32_t want = slices(e + lane, cc);
                        split_write(sq, base, want, (uint32_t)c, qb, cc);
                    }
                } else if (total != 0) {
                    stream(true);
                }
            }
            if ((uint32_t)lane < nq) sq.hits[st + qb + lane] = mycnt;
        }
        const bool is_core = (uint32_t)lane < nq && !((active >> lane) & 1ull);
        if ((uint32_t)lane < nq) core[st + qb + lane] = is_core ? 1 : 0;
        m += (uint32_t)popc64(ballot(is_core));
    }
    if (lane == 0) {
        core_cnt[c] = m;
        if (kSplit && tasks) sq.left[c] = tasks;  // the last of them settles the grid
        if constexpr (kStats) {
            CoreStats& sl = stats[c & (kStatSlots - 1)];
            atomicAdd(&sl.dists, ndist);
            atomicAdd(&sl.points, npts);
            atomicAdd(&sl.grids, ncells);
        }
    }
}

// The tasks core_mark_kernel split off: a wave per task counts the hits of the
// batch's queries that are still open among the task's rows; the wave that
// ends the last task of a grid settles the grid's flags and count.  A stream
// of 3e5 points was 2,300 dependent steps on one wave, while its 150 tasks take
// 16 steps each side by side (2M 2-D points at eps 5000: 1,384 -> 59 + 60 us;
// 3-D at eps 2000: 377 -> 58 + 12 us).
template <int D, bool kStats, bool kPacked, bool kWide>
__global__ __launch_bounds__(kBlock) void core_tasks_kernel(GridView gv, uint8_t* __restrict__ core,
                                                            uint32_t* __restrict__ core_cnt, CoreStats* stats,
                                                            SplitQueue sq) {
    constexpr int PW = packed_words<D>();
    constexpr int QW = kPacked ? PW : D;
    constexpr int S = row_stride(D);
    constexpr int R = 2;
    __shared__ __align__(16) int32_t s_q[kWavesPerBlock][kWave * S];
    const int w = wave_id(), lane = lane_id();
    const uint32_t count = split_used(*sq.count, sq.cap);
    for (uint32_t i = blockIdx.x * kWavesPerBlock + w; i < count; i += gridDim.x * kWavesPerBlock) {
        const uint4 task = sq.tasks[i];
        const uint32_t c = uniform(task.x), qb = uniform(task.y), cc = uniform(task.z);
        if (c == kNone) continue;
        const Inst& I = cell_inst(gv, c);
        const uint32_t st = gv.cell_start[c], k = gv.cell_start[c + 1] - st;
        const uint32_t need = (uint32_t)I.minpts - k;
        const typename Dist<kWide>::T T = inst_T<kWide>(I);
        const uint32_t nq = min((uint32_t)kWave, k - qb);
        const uint32_t row0 = gv.cell_start[cc] + uniform(task.w) * kSplitRows;
        const uint32_t rows = min(kSplitRows, gv.cell_start[cc + 1] - row0);
        const bool valid = (uint32_t)lane < nq;
        const uint32_t s = st + qb + (valid ? lane : 0);
        const uint32_t had = valid ? load_acq(&sq.hits[s]) : need;
        uint64_t active = ballot(had < need);
        {
            int32_t qx[D];
            load_row<D>(gv.crd, s, qx);
            wave_sync();  // the batch before is done with these rows
            if constexpr (kPacked) {
                int32_t pq[PW];
                pack_row<D>(qx, pq);
                store_row<PW>(s_q[w], lane, pq);
            } else {
                store_row<D>(s_q[w], lane, qx);
            }
            wave_sync();
        }
        uint32_t mine = 0;
        unsigned long long ndist = 0, npts = 0;
        int32_t y[R][D];
#pragma unroll
        for (int u = 0; u < R; ++u) load_row<D>(gv.crd, row0 + min((uint32_t)(u * kWave + lane), rows - 1), y[u]);
        for (uint32_t t0 = 0; t0 < rows && active; t0 += R * kWave) {
            int32_t yn[R][D], yp[R][QW];
            uint64_t tvm[R];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                tvm[u] = ballot(t0 + u * kWave + lane < rows);
                load_row<D>(gv.crd, row0 + min(t0 + (uint32_t)((R + u) * kWave + lane), rows - 1), yn[u]);
                if constexpr (kPacked) {
                    pack_row<D>(y[u], yp[u]);
                } else {
#pragma unroll
                    for (int j = 0; j < D; ++j) yp[u][j] = y[u][j];
                }
            }
            const uint64_t act0 = uniform64(active);
            for (uint64_t act = act0; act; act &= act - 1ull) {
                const int qi = ffs64(act);
                int32_t p[QW];
                load_row<QW>(s_q[w], qi, p);
                uint32_t h = 0;
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    if constexpr (kPacked)
                        h += (uint32_t)popc64(ballot(sqdist_pk<D>(yp[u], p) <= T) & tvm[u]);
                    else
                        h += (uint32_t)popc64(ballot(sqdist_nb<D, kWide>(yp[u], p) <= T) & tvm[u]);
                }
                mine += lane == qi ? h : 0u;
                if constexpr (kStats) ndist += min(rows - t0, (uint32_t)(R * kWave));
            }
            if constexpr (kStats) npts += min(rows - t0, (uint32_t)(R * kWave));
            active = act0 & ~ballot(((act0 >> lane) & 1ull) && had + mine >= need);
#pragma unroll
            for (int u = 0; u < R; ++u)
#pragma unroll
                for (int j = 0; j < D; ++j) y[u][j] = yn[u][j];
        }
        if (mine) atomicAdd(&sq.hits[s], mine);
        if constexpr (kStats) {
            if (lane == 0) {
                CoreStats& sl = stats[c & (kStatSlots - 1)];
                atomicAdd(&sl.dists, ndist);
                atomicAdd(&sl.points, npts);
            }
        }
        if (!split_last(sq, c)) continue;
        uint32_t m = 0;
        for (uint32_t q0 = 0; q0 < k; q0 += kWave) {
            const bool in = q0 + lane < k && load_acq(&sq.hits[st + (q0 + lane < k ? q0 + lane : 0)]) >= need;
            if (q0 + lane < k) core[st + q0 + lane] = in ? 1 : 0;
            m += (uint32_t)popc64(ballot(in));
        }
        if (lane == 0) core_cnt[c] = m;
    }
}
// One grid with fewer than MinPts points, marked by S lanes (16: a quarter of a
// wave, 64: all of it) whose first lane is g0.  As core_mark_kernel, with every
// scan, mask and count taken within the group; a step takes two candidates per
// lane.  Returns false, with nothing written, if a group of 16 meets a long
// stream or more points than lanes: those want a whole wave.
template <int S, int D, bool kPacked>
__device__ __forceinline__ bool mark_grid(const GridView& gv, const uint32_t* __restrict__ nei, uint32_t st, uint32_t k,
                                          uint64_t e0, uint64_t e1, uint32_t need, uint32_t T, int g0, int sub,
                                          uint32_t* row, uint32_t* place, int32_t* qrow, uint8_t* __restrict__ core,
                                          uint32_t& m) {
    constexpr int R = 2;
    constexpr int PW = packed_words<D>();
    constexpr int QW = kPacked ? PW : D;
    constexpr uint64_t kAll = S == kWave ? ~0ull : (1ull << (S & 63)) - 1ull;
    auto group = [&](bool x) -> uint64_t { return (ballot(x) >> g0) & kAll; };
    m = 0;
    if (S < kWave && k > (uint32_t)S) return false;
    for (uint32_t qb = 0; qb < k; qb += S) {
        const uint32_t nq = min((uint32_t)S, k - qb);
        uint64_t active = nq == (uint32_t)kWave ? ~0ull : (1ull << nq) - 1ull;
        {
            int32_t qx[D];
            load_row<D>(gv.crd, (uint32_t)sub < nq ? st + qb + sub : st, qx);
            if constexpr (kPacked) {
                int32_t pq[PW];
                pack_row<D>(qx, pq);
                store_row<PW>(qrow, sub, pq);
            } else {
                store_row<D>(qrow, sub, qx);
            }
        }
        uint32_t mycnt = 0;  // lane i of the group: hits of query i
        for (uint64_t e = e0; e < e1 && active; e += S) {
            uint32_t cs = 0, cn = 0;
            if (e + sub < e1) {
                const uint32_t cc = nei[e + sub];
                cs = gv.cell_start[cc];
                cn = gv.cell_start[cc + 1] - cs;
            }
            uint32_t incl = cn;
            if constexpr (S == kWave) {
                incl = wave_incl_scan(incl);
            } else {
                incl += dpp<kRowShr + 1>(0u, incl);
                incl += dpp<kRowShr + 2>(0u, incl);
                incl += dpp<kRowShr + 4>(0u, incl);
                incl += dpp<kRowShr + 8>(0u, incl);
            }
            const uint32_t tot = __shfl(incl, S - 1, S);
            if (S < kWave && tot > kGroupStream) return false;
            row[sub] = cs - (incl - cn);
            place[sub] = incl - cn;
            wave_sync();
            for (uint32_t t0 = 0; t0 < tot && active; t0 += R * S) {
                int32_t y[R][QW];
                bool in[R];
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const uint32_t t = t0 + u * S + sub;
                    in[u] = t < tot;
                    int j = 0;
#pragma unroll
                    for (int step = S / 2; step > 0; step >>= 1)
                        if (place[j + step] <= t) j += step;
                    int32_t x[D];
                    load_row<D>(gv.crd, in[u] ? row[j] + t : st, x);
                    if constexpr (kPacked) {
                        pack_row<D>(x, y[u]);
                    } else {
#pragma unroll
                        for (int d = 0; d < D; ++d) y[u][d] = x[d];
                    }
                }
                uint32_t hits = 0;
                for (uint64_t act = active; act; act &= act - 1ull) {
                    const int q = ffs64(act);
                    int32_t p[QW];
                    load_row<QW>(qrow, q, p);
                    uint32_t h = 0;
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        if constexpr (kPacked)
                            h += (uint32_t)popc64(group(in[u] && sqdist_pk<D>(y[u], p) <= T));
                        else
                            h += (uint32_t)popc64(group(in[u] && sqdist_nb<D, false>(y[u], p) <= T));
                    }
                    hits = sub == q ? h : hits;
                }
                mycnt += hits;
                active &= ~group(mycnt >= need);
            }
            wave_sync();
        }
        const bool is_core = (uint32_t)sub < nq && !((active >> sub) & 1ull);
        if ((uint32_t)sub < nq) core[st + qb + sub] = is_core ? 1 : 0;
        m += (uint32_t)popc64(group(is_core));
    }
    return true;
}

// Marking with 16 lanes per grid, four grids side by side in a wave, for short
// lists and small grids (the rule of the other small-grid kernels): a grid of a
// few noise points with a few neighbours fills a quarter of a wave's lanes at
// best, and the kernel is bound by the instructions and dependent loads of each
// wave.  Grids that want more are taken by the whole wave one after another.
// Lists of 40 and grids of 32 points on
// average: the batch of 256 2,255 -> 1,514 us, 2M 3-D points in small clusters
// 105 -> 58, 1M 2-D noise beside lumps of 1e5 303 -> 109; beside lumps of 2e4 it went
// up to 520 from 390 us before the whole wave took the long streams.  MinPts above
// 32 stays with a wave per grid (60: 368 us there, 671 here).
template <int D, bool kPacked>
__global__ __launch_bounds__(kBlock) void core_mark_group_kernel(GridView gv, const uint64_t* __restrict__ nei_off,
                                                                 const uint32_t* __restrict__ nei,
                                                                 uint8_t* __restrict__ core,
                                                                 uint32_t* __restrict__ core_cnt) {
    constexpr int S = 16, G = kWave / S;
    constexpr int Q = row_stride(kPacked ? packed_words<D>() : D);
    __shared__ uint32_t s_row[kWavesPerBlock][kWave];    // first row of each lane's grid, minus its place
    __shared__ uint32_t s_place[kWavesPerBlock][kWave];  // its place
    __shared__ __align__(16) int32_t s_q[kWavesPerBlock][kWave * Q];
    const int w = wave_id(), lane = lane_id();
    const int grp = lane / S, sub = lane % S, g0 = grp * S;
    const int64_t c = (xcd_runs<16>(block_id(), block_count()) * kWavesPerBlock + w) * G + grp;
    bool whole = false;  // the grid waits for the whole wave
    uint32_t st = 0, k = 0, need = 0, T = 0;
    uint64_t e0 = 0, e1 = 0;
    if (c < (int64_t)*gv.ncell_dev) {
        const Inst& I = cell_inst(gv, c);
        st = gv.cell_start[c];
        k = gv.cell_start[c + 1] - st;
        e0 = nei_off[c];
        e1 = nei_off[c + 1];
        T = I.T;
        if (kPacked && I.eps > kPackedEpsMax) {
            // a replayed graph met a larger eps than it was captured for: the
            // packed differences could wrap, so the run is discarded
            if (sub == 0) atomicOr(&gv.b.hdr->err, kErrPlan);
        } else if (k >= (uint32_t)I.minpts) {
            for (uint32_t i = sub; i < k; i += S) core[st + i] = 1;
            if (sub == 0) core_cnt[c] = k;
        } else {
            need = (uint32_t)I.minpts - k;
            uint32_t m;
            if (mark_grid<S, D, kPacked>(gv, nei, st, k, e0, e1, need, T, g0, sub, &s_row[w][g0], &s_place[w][g0],
                                         &s_q[w][g0 * Q], core, m)) {
                if (sub == 0) core_cnt[c] = m;
            } else {
                whole = true;
            }
        }
    }
    for (uint64_t todo = ballot(whole && sub == 0); todo; todo &= todo - 1ull) {
        const int src = ffs64(todo);
        wave_sync();
        auto lo = [&](uint32_t v) -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)v, src); };
        auto wide = [&](uint64_t v) -> uint64_t { return (uint64_t)lo((uint32_t)(v >> 32)) << 32 | lo((uint32_t)v); };
        uint32_t m;
        mark_grid<kWave, D, kPacked>(gv, nei, lo(st), lo(k), wide(e0), wide(e1), lo(need), lo(T), 0, lane, s_row[w],
                                     s_place[w], s_q[w], core, m);
        if (lane == src) core_cnt[c] = m;
    }
}

// Marking with neighbours as runs (runs.hpp): as core_mark_kernel, but a lane
// owns a run of neighbouring grids, which is one contiguous range of points;
// the own points come with the run of the own family and count like the others.
// The entries that touch lead the list, so most queries close within its first
// chunk: 2M 7-D points (MinPts 100) 1.20 -> 0.32 ms; 10M 5-D points 8.0 -> 8.4 ms,
// the key searches costing what the order saves there (371 vector instructions a
// wave, half the issue rate).  A wave for several grids of a family at a time was
// slower (14.6 ms: wider windows, and every wave waits for its slowest query).
template <int D, bool kPacked, int R>
__global__ __launch_bounds__(kBlock) void core_mark_runs_kernel(GridView gv, RunSource rs, uint8_t* __restrict__ core,
                                                                uint32_t* __restrict__ core_cnt) {
    constexpr int PW = packed_words<D>();
    constexpr int QW = kPacked ? PW : D;
    constexpr int S = row_stride(D);
    __shared__ uint32_t s_row[kWavesPerBlock][kWave];   // first row of each lane's run, minus its place
    __shared__ uint32_t s_head[kWavesPerBlock][kWave];  // lane + 1 of the run that starts at this candidate
    __shared__ __align__(16) int32_t s_q[kWavesPerBlock][kWave * S];  // the query rows of the batch
    const int w = wave_id(), lane = lane_id();
    const int64_t c = xcd_runs<16>(block_id(), block_count()) * kWavesPerBlock + w;
    if (c >= (int64_t)*gv.ncell_dev) return;
    const Inst& I = cell_inst(gv, c);
    const uint32_t st = gv.cell_start[c];
    const uint32_t en = gv.cell_start[c + 1];
    RunCursor<D> rc;
    rc.open(rs, gv, c);
    const uint32_t minpts = (uint32_t)I.minpts;
    const uint32_t T = I.T;
    const uint32_t k = en - st;
    if (kPacked && I.eps > kPackedEpsMax) {
        // a replayed graph met a larger eps than it was captured for: the
        // packed differences could wrap, so the run is discarded
        if (lane == 0) atomicOr(&gv.b.hdr->err, kErrPlan);
        return;
    }
    if (k >= minpts) {
        for (uint32_t i = lane; i < k; i += kWave) core[st + i] = 1;
        if (lane == 0) core_cnt[c] = k;
        return;
    }
    uint32_t m = 0;
    for (uint32_t qb = 0; qb < k; qb += kWave) {
        const uint32_t nq = min((uint32_t)kWave, k - qb);
        uint64_t active = nq == (uint32_t)kWave ? ~0ull : ((1ull << nq) - 1ull);
        {
            int32_t qx[D];
            load_row<D>(gv.crd, (uint32_t)lane < nq ? st + qb + lane : st, qx);
            if constexpr (kPacked) {
                int32_t pq[PW];
                pack_row<D>(qx, pq);
                store_row<PW>(s_q[w], lane, pq);
            } else {
                store_row<D>(s_q[w], lane, qx);
            }
        }
        uint32_t mycnt = 0;  // lane i: hits of query i
        for (uint64_t e = rc.e0; e < rc.e1 && active; e += kWave) {
            uint32_t lo = 0, hi = 0;
            if (e + lane < rc.e1) rc.run_of(rs, rs.ent[e + lane], lo, hi);
            const uint32_t cs = lo < hi ? gv.cell_start[lo] : 0u;
            const uint32_t cn = lo < hi ? gv.cell_start[hi] - cs : 0u;
            const uint32_t incl = wave_incl_scan(cn);
            const uint32_t tot = last_lane(incl);
            const uint32_t excl = incl - cn;
            s_row[w][lane] = cs - excl;
            // Row of flat candidate t0 + lane: the runs that start within the
            // step mark their first candidate, a running maximum over the lanes
            // gives each candidate its run, and the last one carries over to
            // the next step.
            uint32_t carry = 0;
            auto cand_row = [&](uint32_t t0) -> uint32_t {
                s_head[w][lane] = 0;
                wave_sync();
                if (cn != 0 && excl >= t0 && excl < t0 + kWave) s_head[w][excl - t0] = (uint32_t)lane + 1u;
                wave_sync();
                uint32_t own = wave_max_scan(s_head[w][lane]);
                own = own ? own : carry;
                carry = last_lane(own);
                return s_row[w][(own ? own : 1u) - 1u] + t0 + lane;
            };
            int32_t y[R][D];
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const uint32_t t = (uint32_t)(u * kWave);
                const uint32_t r = cand_row(t);
                load_row<D>(gv.crd, t + lane < tot ? r : st, y[u]);
            }
            for (uint32_t t0 = 0; t0 < tot && active; t0 += R * kWave) {
                uint64_t tvm[R];
#pragma unroll
                for (int u = 0; u < R; ++u) tvm[u] = ballot(t0 + u * kWave + lane < tot);
                int32_t yn[R][D];
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const uint32_t t = t0 + (R + u) * kWave;
                    uint32_t r = st;
                    if (t < tot) r = cand_row(t);
                    load_row<D>(gv.crd, t + lane < tot ? r : st, yn[u]);
                }
                int32_t yp[R][QW];
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    if constexpr (kPacked) {
                        pack_row<D>(y[u], yp[u]);
                    } else {
#pragma unroll
                        for (int j = 0; j < D; ++j) yp[u][j] = y[u][j];
                    }
                }
                const uint64_t act0 = uniform64(active);
                uint32_t step_hits = 0;
                for (uint64_t act = act0; act;) {
                    const int qa = ffs64(act);
                    act &= act - 1ull;
                    const int qc = act ? ffs64(act) : qa;
                    act &= act - 1ull;
                    uint32_t ha = 0, hc = 0;
                    int32_t pa[QW], pc[QW];
                    load_row<QW>(s_q[w], qa, pa);
                    load_row<QW>(s_q[w], qc, pc);
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        if constexpr (kPacked) {
                            ha += (uint32_t)popc64(ballot(sqdist_pk<D>(yp[u], pa) <= T) & tvm[u]);
                            hc += (uint32_t)popc64(ballot(sqdist_pk<D>(yp[u], pc) <= T) & tvm[u]);
                        } else {
                            ha += (uint32_t)popc64(ballot(sqdist_nb<D, false>(yp[u], pa) <= T) & tvm[u]);
                            hc += (uint32_t)popc64(ballot(sqdist_nb<D, false>(yp[u], pc) <= T) & tvm[u]);
                        }
                    }
                    step_hits = lane == qa ? ha : step_hits;
                    step_hits = lane == qc ? hc : step_hits;
                }
                mycnt += step_hits;
                active = act0 & ~ballot(((act0 >> lane) & 1ull) && mycnt >= minpts);
#pragma unroll
                for (int u = 0; u < R; ++u)
#pragma unroll
                    for (int j = 0; j < D; ++j) y[u][j] = yn[u][j];
            }
            wave_sync();
        }
        const bool is_core = (uint32_t)lane < nq && !((active >> lane) & 1ull);
        if ((uint32_t)lane < nq) core[st + qb + lane] = is_core ? 1 : 0;
        m += (uint32_t)popc64(ballot(is_core));
    }
    if (lane == 0) core_cnt[c] = m;
}

template <bool kStats, bool kPacked, int R, bool kWide>
hipError_t launch_core_mark_as(const GridView& g, const uint64_t* nei_off, const uint32_t* nei, const uint2* mid,
                               uint8_t* core, uint32_t* core_cnt, CoreStats* stats, const SplitQueue* split,
                               hipStream_t st) {
    const unsigned blocks = grid_for(g.ncell, kWavesPerBlock);
    if (split)
        GD_DISPATCH_D(g.D, ({
                          core_mark_kernel<D, kStats, kPacked, R, kWide, true><<<grid_of(blocks), dim3(kBlock), 0, st>>>(
                              g, nei_off, nei, mid, core, core_cnt, stats, *split);
                          core_tasks_kernel<D, kStats, kPacked, kWide>
                              <<<dim3(kSplitBlocks), dim3(kBlock), 0, st>>>(g, core, core_cnt, stats, *split);
                      }));
    else
        GD_DISPATCH_D(g.D, (core_mark_kernel<D, kStats, kPacked, R, kWide, false>
                            <<<grid_of(blocks), dim3(kBlock), 0, st>>>(g, nei_off, nei, mid, core, core_cnt, stats,
                                                                       SplitQueue{})));
    return hipGetLastError();
}

template <bool kPacked, int R>
hipError_t launch_core_mark_runs(const GridView& g, const RunSource& rs, uint8_t* core, uint32_t* core_cnt,
                                 hipStream_t st) {
    const unsigned blocks = grid_for(g.ncell, kWavesPerBlock);
    GD_DISPATCH_D(g.D, ({
                      if constexpr (D >= kMinRunD) {
                          core_mark_runs_kernel<D, kPacked, R>
                              <<<grid_of(blocks), dim3(kBlock), 0, st>>>(g, rs, core, core_cnt);
                          return hipGetLastError();
                      }
                  }));
    return hipErrorInvalidValue;
}

hipError_t launch_core_mark(const GridView& g, const uint64_t* nei_off, const uint32_t* nei, const uint2* mid,
                            const RunSource* runs,
                            uint8_t* core, uint32_t* core_cnt, CoreStats* stats, int64_t max_eps, int64_t min_minpts,
                            const SplitQueue* split, int lanes, hipStream_t st) {
    if (g.ncell == 0) return hipSuccess;
    const bool packed = core_mark_packed(max_eps);
    const bool two = min_minpts > kWave / 2;
    if (runs) {
        if (stats || split || max_eps > GD_EPS_MAX) return hipErrorInvalidValue;
        if (packed && two) return launch_core_mark_runs<true, 2>(g, *runs, core, core_cnt, st);
        if (packed) return launch_core_mark_runs<true, 1>(g, *runs, core, core_cnt, st);
        if (two) return launch_core_mark_runs<false, 2>(g, *runs, core, core_cnt, st);
        return launch_core_mark_runs<false, 1>(g, *runs, core, core_cnt, st);
    }
    if (lanes == 16 && !two && !stats && !split && max_eps <= GD_EPS_MAX) {
        const dim3 blocks = grid_of((g.ncell + 4 * kWavesPerBlock - 1) / (4 * kWavesPerBlock));
        if (packed)
            GD_DISPATCH_D(g.D, (core_mark_group_kernel<D, true><<<blocks, dim3(kBlock), 0, st>>>(g, nei_off, nei, core,
                                                                                               core_cnt)));
        else
            GD_DISPATCH_D(g.D, (core_mark_group_kernel<D, false><<<blocks, dim3(kBlock), 0, st>>>(g, nei_off, nei, core,
                                                                                                core_cnt)));
        return hipGetLastError();
    }
    // the counting variant takes the same steps as the timed one (of a wave per grid)
    auto mark = [&](auto launch) { return launch(g, nei_off, nei, mid, core, core_cnt, stats, split, st); };
    if (max_eps > GD_EPS_MAX) {  // 64-bit distances, one row per step
        return stats ? mark(launch_core_mark_as<true, false, 1, true>)
                     : mark(launch_core_mark_as<false, false, 1, true>);
    }
    if (stats)
        return two ? mark(launch_core_mark_as<true, false, 2, false>)
                   : mark(launch_core_mark_as<true, false, 1, false>);
    if (packed)
        return two ? mark(launch_core_mark_as<false, true, 2, false>)
                   : mark(launch_core_mark_as<false, true, 1, false>);
    return two ? mark(launch_core_mark_as<false, false, 2, false>)
               : mark(launch_core_mark_as<false, false, 1, false>);
}

// Side rows of grid c: its core count if it also holds non-core points.
struct SideRows {
    const uint32_t* cnt;
    const uint32_t* cell_start;
    const uint32_t* ncell;
    __device__ uint32_t operator()(int64_t c) const {
        if (c >= (int64_t)*ncell) return 0u;
        const uint32_t m = cnt[c];
        return (m != 0 && m != cell_start[c + 1] - cell_start[c]) ? m : 0u;
    }
};

// One thread per grid: where its core set starts, the smallest input index
// of its core points (grids without side rows), and the header counts.  The
// counts are reduced per workgroup and written to part[] (five words per
// workgroup), then summed by core_counts_fold: atomics from every wave to
// five addresses serialise on grids by the million.
__global__ __launch_bounds__(kBlock) void core_cells_kernel(GridView gv, CoreOut co, uint32_t* part) {
    __shared__ uint32_t red[5][kWavesPerBlock];
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool v = c < (int64_t)*gv.ncell_dev;
    uint32_t cnt = 0, size = 0, minpts = 0;
    if (v) {
        const uint32_t st = gv.cell_start[c];
        cnt = co.core_cnt[c];
        size = gv.cell_start[c + 1] - st;
        minpts = (uint32_t)cell_inst(gv, c).minpts;
        const bool side = cnt != 0 && cnt != size;
        co.core_begin[c] = side ? (uint32_t)gv.n + co.side_off[c] : st;
        if (!side) co.cell_min_core[c] = cnt ? gv.sidx[st] : kNone;
    }
    const uint32_t has = (uint32_t)popc64(ballot(v && cnt > 0));
    const uint32_t dense = (uint32_t)popc64(ballot(v && size >= minpts));
    const uint32_t tiny = (uint32_t)popc64(ballot(v && cnt > 0 && cnt <= kTinyCore));
    const uint32_t mx = wave_max_u32(cnt);
    const uint32_t tot = wave_sum(cnt);
    const int w = wave_id();
    if (lane_id() == 0) {
        red[0][w] = tot;
        red[1][w] = has;
        red[2][w] = mx;
        red[3][w] = dense;
        red[4][w] = tiny;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        uint32_t a = 0;
        for (int ww = 0; ww < kWavesPerBlock; ++ww)
            a = threadIdx.x == 2 ? max(a, red[2][ww]) : a + red[threadIdx.x][ww];
        part[(int64_t)blockIdx.x * 5 + threadIdx.x] = a;
    }
}

// counts[0..4] from the per-workgroup words of core_cells_kernel, by one
// workgroup (the first of the side copy, which needs no extra launch).
__device__ __forceinline__ void core_counts_fold(const uint32_t* part, int64_t blocks, uint32_t* counts) {
    __shared__ uint32_t red[5][kWavesPerBlock];
    uint32_t a[5] = {0, 0, 0, 0, 0};
    for (int64_t b = threadIdx.x; b < blocks; b += kBlock) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const uint32_t x = part[b * 5 + k];
            a[k] = k == 2 ? max(a[k], x) : a[k] + x;
        }
    }
    const int w = wave_id();
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const uint32_t r = k == 2 ? wave_max_u32(a[k]) : wave_sum(a[k]);
        if (lane_id() == 0) red[k][w] = r;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        uint32_t r = 0;
        for (int ww = 0; ww < kWavesPerBlock; ++ww)
            r = threadIdx.x == 2 ? max(r, red[2][ww]) : r + red[threadIdx.x][ww];
        counts[threadIdx.x] = r;
    }
}

// One wave per grid holding both core and non-core points: copy its core
// rows, in sorted order, to the side area.  Workgroup 0 first folds the
// header counts (part, blocks: see core_cells_kernel).
template <int D>
__global__ __launch_bounds__(kBlock) void side_copy_kernel(GridView gv, CoreOut co, const uint32_t* part,
                                                           int64_t blocks) {
    if (blockIdx.x == 0) core_counts_fold(part, blocks, co.counts);
    // each wave checks 64 grids at once (one lane each) and copies only the
    // mixed ones: most grids need nothing, and a wave launched per grid would
    // spend the kernel on dispatching waves that exit at once
    const int lane = lane_id();
    const int64_t c0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave_id()) * kWave;
    const int64_t ncell = *gv.ncell_dev;
    const int64_t cl = c0 + lane;
    uint32_t st_l = 0, k_l = 0, m_l = 0;
    if (cl < ncell) {
        st_l = gv.cell_start[cl];
        k_l = gv.cell_start[cl + 1] - st_l;
        m_l = co.core_cnt[cl];
    }
    uint64_t todo = ballot(cl < ncell && m_l != 0 && m_l != k_l);
    while (todo) {
        const int g = ffs64(todo);
        todo &= todo - 1ull;
        const int64_t c = c0 + g;
        const uint32_t st = readlane(st_l, g), k = readlane(k_l, g);
        const uint32_t base = (uint32_t)gv.n + co.side_off[c];
        uint32_t done = 0, first = kNone;
        for (uint32_t qb = 0; qb < k; qb += kWave) {
            const bool v = qb + lane < k;
            const bool f = v && co.core[st + qb + lane];
            const uint32_t orig = v ? gv.sidx[st + qb + lane] : 0u;
            const uint64_t bal = ballot(f);
            if (f) {
                const uint32_t r = base + done + (uint32_t)popc64(bal & lanemask_lt());
                int32_t y[D];
                load_row<D>(gv.crd, st + qb + lane, y);
                store_row<D>(co.ccrd, r, y);
                co.corig[r] = orig;
            }
            // sorted order within a grid is input order: the first core point has the smallest index
            if (first == kNone && bal) first = readlane(orig, ffs64(bal));
            done += (uint32_t)popc64(bal);
        }
        if (lane == 0) co.cell_min_core[c] = first;
    }
}

hipError_t launch_core_compact(const GridView& g, const CoreOut& c, uint32_t* partial, hipStream_t st) {
    if (g.ncell == 0) return fill<uint32_t>(c.counts, 5, 0u, st);
    hipError_t e;
    e = scan_exclusive<uint32_t>(SideRows{c.core_cnt, g.cell_start, g.ncell_dev}, g.ncell + 1, c.side_off,
                                 (uint32_t*)nullptr, partial, st);
    if (e != hipSuccess) return e;
    const unsigned nb = grid_for(g.ncell);
    core_cells_kernel<<<dim3(nb), dim3(kBlock), 0, st>>>(g, c, c.count_part);
    GD_DISPATCH_D(g.D, (side_copy_kernel<D><<<dim3(grid_for(g.ncell, kWavesPerBlock * kWave)), dim3(kBlock), 0, st>>>(
                           g, c, c.count_part, (int64_t)nb)));
    return hipGetLastError();
}

struct CoreCellFlag {
    const uint32_t* core_cnt;
    const uint32_t* ncell;
    __device__ uint32_t operator()(int64_t c) const { return c < (int64_t)*ncell && core_cnt[c] > 0; }
};

// Output of the core-grid scan: the list of core grids (and their counts as
// sort keys) in grid order, the merge record reset, every grid its own
// union-find root, and the per-root minima of the labelling step cleared.
struct CoreListWriter {
    const uint32_t* ncell;
    const uint32_t* core_cnt;
    uint32_t* list;
    uint32_t* keys;
    uint4* rec;
    uint32_t* parent;
    uint32_t* root_min;
    __device__ void operator()(int64_t c, uint32_t ex, uint32_t is_core) const {
        if (c >= (int64_t)*ncell) return;
        rec[c] = make_uint4(kNone, 0u, 0u, 0u);
        parent[c] = (uint32_t)c;
        root_min[c] = kNone;
        if (is_core) {
            list[ex] = (uint32_t)c;
            keys[ex] = core_cnt[c];
        }
    }
};

// The merge step's record of each core grid: rank in the visiting order,
// first row and size of its core set (one load instead of three).
__global__ __launch_bounds__(kBlock) void rank_kernel(const uint32_t* sorted, const uint32_t* m, CoreOut co,
                                                      uint4* rec) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= (int64_t)*m) return;
    const uint32_t c = sorted[r];
    rec[c] = make_uint4((uint32_t)r, co.core_begin[c], co.core_cnt[c], 0u);
}

hipError_t launch_ldf_order(const GridView& g, const CoreOut& c, bool by_count, int64_t ncc, int count_bits,
                            bool pad_tail, uint32_t* list, uint4* rank, uint32_t* parent, uint32_t* root_min,
                            uint32_t* keys_a, uint32_t* keys_b, uint32_t* vals_b, uint32_t* radix_scratch,
                            uint32_t* partial, uint32_t** sorted_list, hipStream_t st) {
    *sorted_list = list;
    if (g.ncell == 0) return hipSuccess;
    if (by_count && pad_tail && ncc > 0) {
        hipError_t e = fill<uint32_t>(keys_a, ncc, (uint32_t)((1ull << count_bits) - 1ull), st);
        if (e != hipSuccess) return e;
    }
    hipError_t e = scan_apply<uint32_t>(CoreCellFlag{c.core_cnt, g.ncell_dev}, g.ncell,
                                        CoreListWriter{g.ncell_dev, c.core_cnt, list, keys_a, rank, parent, root_min},
                                        (uint32_t*)nullptr, partial, st);
    if (e != hipSuccess) return e;
    if (by_count && ncc > 1) {
        RadixResult<uint32_t> res;
        e = radix_sort_pairs<uint32_t>(keys_a, list, keys_b, vals_b, ncc, count_bits, false, radix_scratch, st, &res);
        if (e != hipSuccess) return e;
        *sorted_list = res.vals;
    }
    if (ncc > 0) rank_kernel<<<dim3(grid_for(ncc)), dim3(kBlock), 0, st>>>(*sorted_list, &c.counts[1], c, rank);
    return hipGetLastError();
}

}  // namespace gd
