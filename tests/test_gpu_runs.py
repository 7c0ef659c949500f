"""Sparse data: neighbours as runs of grids below the entries of a family's
node list (four dimensions and more, the default), and the lists of two and
three dimensions built level by level, against the oracle and against the
lists written per grid (GD_OPT_NEIGHBOR_MODE = 1)."""
import numpy as np
import pytest

import oracle
import workloads as W
from oracle import steps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    import paper_2210_07580_amd as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return G


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def check(G, x, eps, minpts, options=()):
    ctx = G.Context(0)
    for k, v in options:
        ctx.set_option(k, v)
    lab, core = ctx.dbscan(dev(x), eps, minpts)
    want = oracle.dbscan(x, eps, minpts)
    assert np.array_equal(core.cpu().numpy(), want[1])
    assert np.array_equal(lab.cpu().numpy(), want[0])
    return ctx


def uniform(seed, n, d, domain):
    return np.random.default_rng(seed).integers(0, domain, size=(n, d)).astype(np.int32)


# few and many points per neighbourhood, one point up to several waves' worth
@pytest.mark.parametrize("d", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("n,domain,eps,minpts", [(1, 10, 3, 1), (65, 60, 20, 2), (700, 300, 90, 4),
                                                 (6000, 1000, 260, 9), (6000, 400, 150, 40)])
def test_uniform(G, d, n, domain, eps, minpts):
    print(f"case d={d} n={n}", flush=True)
    check(G, uniform(d * 100 + n, n, d, domain), eps, minpts).close()


@pytest.mark.parametrize("d", [4, 5, 8])
def test_long_families(G, d):
    # hundreds of grids share all keys but the last (64-grid slices and binary
    # searches over long rows), in two rows next to each other, plus noise
    rng = np.random.default_rng(d)
    m = 3000
    x = np.zeros((2 * m, d), np.int32)
    x[:, -1] = rng.integers(0, 60_000, size=2 * m)
    x[m:, 0] = 70
    x = np.concatenate([x, rng.integers(0, 60_000, size=(500, d)).astype(np.int32)])
    check(G, x, 100, 3).close()


@pytest.mark.parametrize("eps", [9_000, 12_000, 21_845, 22_000])
def test_distance_widths(G, eps):
    # packed 16-bit differences, 32-bit, and the 64-bit path (which keeps lists)
    x = uniform(eps, 4000, 5, 6 * eps)
    check(G, x, eps, 5).close()


def test_heavy_core_sets(G):
    # two grids of 9000 points within eps of each other among sparse ones: their
    # pair goes to the queue for whole workgroups
    rng = np.random.default_rng(5)
    a = rng.integers(0, 40, size=(9000, 4)) + 5000
    b = rng.integers(0, 40, size=(9000, 4)) + np.array([5090, 5000, 5000, 5000])
    x = np.concatenate([a, b, rng.integers(0, 10_000, size=(20_000, 4))]).astype(np.int32)
    check(G, x[rng.permutation(len(x))], 100, 20).close()


def test_lists_and_counts_on_request(G):
    # the default writes no lists at d >= 4: the count and the debug view give
    # what the list mode gives
    w = W.WORKLOADS["cfg2"].with_n(30_000)
    x = W.make_points(w)
    runs = check(G, x, w.eps, w.minpts)
    lists = check(G, x, w.eps, w.minpts, [(G.GD_OPT_NEIGHBOR_MODE, 1)])
    assert runs.stats()["neighbor_entries"] == lists.stats()["neighbor_entries"]
    assert runs.stats() == lists.stats()
    for got, want in zip(runs.debug_neighbors(), lists.debug_neighbors()):
        assert np.array_equal(got, want)
    runs.close()
    lists.close()


@pytest.mark.parametrize("d", [2, 3])
def test_level_lists_are_in_walk_order(G, d):
    x = uniform(d, 3000, d, 900)
    ctx = check(G, x, 40, 3, [(G.GD_OPT_NEIGHBOR_QUERY, 1)])
    _, _, ids = ctx.debug_grids()
    off, nei = ctx.debug_neighbors()
    want, _ = steps.neighbor_grids(ids)
    turn = {0: 0, 1: 1, 2: 2, 3: 3, -1: 4, -2: 5, -3: 6}
    for g in range(len(ids)):
        got = nei[off[g]:off[g + 1]].astype(np.int64)
        order = sorted(want[g].tolist(), key=lambda h: (turn[int(ids[h][0] - ids[g][0])], h))
        assert got.tolist() == order, f"grid {g}"
    ctx.close()


def batch(seed, scale=1):
    rng = np.random.default_rng(seed)
    out = []
    for k in range(12):
        d = int(rng.integers(2, 7)) if k else 6
        n = int(rng.integers(200, 2500)) * scale
        out.append((rng.integers(0, 500, size=(n, d)).astype(np.int32), int(rng.integers(60, 160)),
                    int(rng.integers(2, 12))))
    return out


def test_batch_of_mixed_dimensions_replayed(G):
    # instances of fewer dimensions than the batch's largest; replays with other
    # data of the same shape, then with data that outgrow the plan
    ctx = G.Context(0)
    rng = np.random.default_rng(1)
    first = batch(3)
    for rep in range(4):
        if rep < 3:
            probs = [(rng.integers(0, 500, size=x.shape).astype(np.int32), e, m) for x, e, m in first]
        else:  # one lump: far longer lists than planned for
            probs = [(rng.integers(0, 60, size=x.shape).astype(np.int32), max(e // 20, 2), m) for x, e, m in first]
        outs = ctx.dbscan_batched([(dev(x), e, m) for x, e, m in probs])
        for k, ((lab, core), (x, e, m)) in enumerate(zip(outs, probs)):
            want = oracle.dbscan(x, e, m)
            assert np.array_equal(core.cpu().numpy(), want[1]), f"replay {rep} instance {k}"
            assert np.array_equal(lab.cpu().numpy(), want[0]), f"replay {rep} instance {k}"
        replayed = ctx.stats()["graph_replays"]
        assert replayed == (1 if rep in (1, 2) else 0) or rep == 3
    ctx.close()


def test_limits_and_options_keep_their_paths(G):
    # a workspace limit, stats, the BFS order and the walk mode on the same data
    x = uniform(11, 5000, 5, 700)
    want = check(G, x, 200, 6)
    entries = want.stats()["neighbor_entries"]
    for opts in ([(G.GD_OPT_WORKSPACE_LIMIT, 1 << 30)], [(G.GD_OPT_STATS, 1)], [(G.GD_OPT_MERGE_ORDER, 2)],
                 [(G.GD_OPT_MERGE_ORDER, 0)], [(G.GD_OPT_NEIGHBOR_QUERY, 1)], [(G.GD_OPT_GRAPH, 2)]):
        ctx = check(G, x, 200, 6, opts)
        assert ctx.stats()["neighbor_entries"] == entries, opts
        ctx.close()
    check(G, x, 200, 6, [(G.GD_OPT_NEIGHBOR_MODE, 2)]).close()
    lab = torch.empty(len(x), dtype=torch.int32, device="cuda")
    core = torch.empty(len(x), dtype=torch.uint8, device="cuda")
    want.dbscan_noalloc(dev(x), 200, 6, lab, core)
    ref = oracle.dbscan(x, 200, 6)
    assert np.array_equal(lab.cpu().numpy(), ref[0]) and np.array_equal(core.cpu().numpy(), ref[1])
    assert want.stats()["neighbor_entries"] == entries
    want.close()


@pytest.mark.parametrize("d,cells", [(4, 5), (5, 4), (6, 3)])
@pytest.mark.parametrize("minpts", [4, 30])
def test_dense_grids_from_four_dimensions(G, d, cells, minpts):
    # about twenty points per grid: lists by offset built level by level, and
    # (from five dimensions on) the big-set merge in two launches
    side = 50.0
    n = 20 * cells ** d
    x = uniform(d, n, d, int(cells * side))
    eps = int(side * np.sqrt(d)) + 1
    ctx = check(G, x, eps, minpts, [(G.GD_OPT_NEIGHBOR_MODE, 1)])
    assert ctx.stats()["core_grids"] >= 512 and n >= 8 * ctx.stats()["grids"]
    _, _, ids = ctx.debug_grids()
    off, nei = ctx.debug_neighbors()
    want, _ = steps.neighbor_grids(ids)
    for g in range(0, len(ids), max(1, len(ids) // 60)):
        got = nei[off[g]:off[g + 1]].astype(np.int64)
        order = sorted(want[g].tolist(), key=lambda h: (steps.grid_offset(ids[g], ids[h]), h))
        assert got.tolist() == order, f"grid {g}"
    ctx.close()
    check(G, x, eps, minpts, [(G.GD_OPT_GRAPH, 2)]).close()
