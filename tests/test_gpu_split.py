"""Few grids of thousands of points: core marking and the border search hand the
streams through large neighbours out as tasks (grids of kSplitMean = 256 points
and more on average, slices of 2048 rows), against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    import paper_2210_07580_amd as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return G


def check(G, x, eps, minpts, options=(), calls=1):
    ctx = G.Context(0)
    for k, v in options:
        ctx.set_option(k, v)
    t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()
    want = oracle.dbscan(x, eps, minpts)
    for call in range(calls):
        lab, core = ctx.dbscan(t, eps, minpts)
        assert np.array_equal(core.cpu().numpy(), want[1]), f"call {call}"
        assert np.array_equal(lab.cpu().numpy(), want[0]), f"call {call}"
    st = ctx.stats()
    ctx.close()
    return st


def lumps(seed, d, sizes, eps, around):
    """Lumps of the given sizes one grid apart or two along a line, and `around`
    points spread over their surroundings (in sparse grids next to them); a
    point at the origin puts each lump inside one grid."""
    rng = np.random.default_rng(seed)
    side = eps / np.sqrt(d)
    parts = []
    for i, m in enumerate(sizes):
        lo = np.full(d, 10.05 * side)
        lo[0] += 2.0 * side * i
        parts.append(lo + rng.random((m, d)) * side * 0.9)
    parts.append(10 * side + (rng.random((around, d)) * 2 - 1) * side * 4 + np.eye(1, d)[0] * side * len(sizes))
    parts.append(np.zeros((1, d)))
    x = np.maximum(np.rint(np.concatenate(parts)), 0).astype(np.int32)
    return x[rng.permutation(len(x))]


# sizes around a slice (2048 rows) and several of them
@pytest.mark.parametrize("d,around", [(1, 6), (2, 10), (3, 10), (5, 10), (7, 10)])
@pytest.mark.parametrize("sizes", [(2047, 2048), (2049, 4096), (4097, 2048, 6500)])
@pytest.mark.parametrize("minpts", [3, 700])
def test_slices(G, d, around, sizes, minpts):
    print(f"case d={d} sizes={sizes} minpts={minpts}", flush=True)
    x = lumps(d + len(sizes), d, sizes, 1000, around)
    st = check(G, x, 1000, minpts)
    assert st["n"] >= 256 * st["grids"]


def test_many_queries_per_sparse_grid(G):
    # sparse grids of more than 64 points (several batches of queries) next to
    # large ones, with MinPts above their size: some core, some border, some noise
    rng = np.random.default_rng(3)
    big = rng.random((9000, 2)) * 600
    ring = rng.random((400, 2)) * 700 + np.array([710.0, 0.0])
    far = rng.random((150, 2)) * 700 + np.array([2130.0, 0.0])
    x = np.rint(np.concatenate([big, ring, far])).astype(np.int32)
    for minpts in (200, 500, 3000):
        check(G, x[rng.permutation(len(x))], 1000, minpts)


@pytest.mark.parametrize("eps", [9_000, 15_000, 30_000])
def test_distance_widths(G, eps):
    check(G, lumps(1, 3, (2500, 5000), eps, 14), eps, 300)


def test_counting_replay_and_orders(G):
    x = lumps(2, 2, (5000, 2100, 3000), 800, 14)
    plain = check(G, x, 800, 50)
    counted = check(G, x, 800, 50, [(G.GD_OPT_STATS, 1)])
    assert counted["core_distances"] > 0 and counted["core_points"] == plain["core_points"]
    assert check(G, x, 800, 50, [(G.GD_OPT_GRAPH, 2)], calls=4)["graph_replays"] == 1
    for order in (0, 2):
        check(G, x, 800, 50, [(G.GD_OPT_MERGE_ORDER, order)])
    check(G, x, 800, 50, [(G.GD_OPT_NEIGHBOR_QUERY, 2)])
