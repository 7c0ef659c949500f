"""The merge of big core sets in two launches (768 to 8192 of them in four
dimensions and more): just below, at and beyond both ends, beside tiny sets,
eager and replayed with more and fewer such grids than planned for, against
the oracle."""
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


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def blocks(seed, d, big, small, n=0):
    """`big` grids of 9 points and `small` of 3 (side 50), along a lattice with
    every seventh place left empty; topped up to n points in the first grid."""
    rng = np.random.default_rng(seed)
    total = big + small
    edge = int(np.ceil((total * 1.2 + 8) ** (1 / d)))
    place = [p for p in range(edge ** d) if p % 7 != 3][:total]
    counts = rng.permutation(np.concatenate([np.full(big, 9), np.full(small, 3)]))
    at = np.repeat(np.array(place), counts)
    if n:
        at = np.concatenate([at, np.full(n - len(at), at[0])])
    x = 10 + rng.random((len(at), d)) * 29  # (clear of the cells' edges: eps / sqrt(d) is not quite 50)
    for j in range(d):
        x[:, j] += 50 * (at // edge ** j % edge)
    x = np.floor(np.concatenate([np.zeros((1, d)), x])).astype(np.int32)
    return x[rng.permutation(len(x))]


def check(ctx, x, eps, minpts, want=None):
    want = want or oracle.dbscan(x, eps, minpts)
    lab, core = ctx.dbscan(dev(x), eps, minpts)
    assert np.array_equal(core.cpu().numpy(), want[1])
    assert np.array_equal(lab.cpu().numpy(), want[0])


@pytest.mark.parametrize("d", [4, 5, 7])
@pytest.mark.parametrize("big", [767, 768, 769, 2500, 8192, 8193])
def test_ends_of_the_range(G, d, big):
    print(f"case d={d} big={big}", flush=True)
    ctx = G.Context(0)
    x, eps = blocks(big + d, d, big, 200), int(50 * np.sqrt(d))
    want = oracle.dbscan(x, eps, 3)
    for mode in (0, 1):
        ctx.set_option(G.GD_OPT_NEIGHBOR_MODE, mode)
        check(ctx, x, eps, 3, want)
        assert big <= ctx.stats()["core_grids"] <= big + 200 + 1
    ctx.close()


def test_replays_with_more_and_fewer_big_grids(G):
    d, eps = 5, int(50 * np.sqrt(5))
    n = 9 * 900 + 3 * 700 + 2000
    ctx = G.Context(0)
    ctx.set_option(G.GD_OPT_GRAPH, 2)
    replays = 0
    for big, small in ((900, 700), (900, 700), (940, 640), (1, 900), (900, 0)):
        check(ctx, blocks(big, d, big, small, n), eps, 3)
        replays += ctx.stats()["graph_replays"]
    assert replays >= 3
    ctx.close()
