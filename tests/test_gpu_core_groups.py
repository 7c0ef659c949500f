"""Core marking with 16 lanes per grid: grids of more points than lanes, streams
on both sides of the hand-over to the whole wave, MinPts on both sides of the
rule, packed and plain distances."""
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


def spread(rng, d, eps, lump):
    """Lone points, pairs, grids of 15 to 33 points and lumps around the given size, a cell wide each."""
    side = eps / np.sqrt(d)
    ext = 24 if d == 2 else 9 if d == 3 else 4
    cells = rng.integers(0, ext, size=(260, d))
    sizes = np.resize([1, 1, 2, 1, 15, 1, 16, 17, 1, 31, 32, 33, 1, lump - 1, lump, lump + 1], len(cells))
    x = np.repeat(cells, sizes, axis=0) * side + rng.random((sizes.sum(), d)) * side
    return np.rint(x).astype(np.int32)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("eps", [60, 10_000, 10_001, 21_845])
@pytest.mark.parametrize("minpts,lump", [(2, 20), (18, 128), (32, 256), (32, 3), (33, 100)])
def test_core_groups(G, d, eps, minpts, lump):
    x = spread(np.random.default_rng(d * 100 + minpts), d, eps, lump)
    ctx = G.Context(0)
    ctx.set_option(G.GD_OPT_GRID_LANES, 16)
    lab, core = ctx.dbscan(torch.from_numpy(x.astype(np.float32)).cuda(), eps, minpts)
    want = oracle.dbscan(x, eps, minpts)
    ctx.close()
    assert np.array_equal(core.cpu().numpy(), want[1])
    assert np.array_equal(lab.cpu().numpy(), want[0])


def test_core_groups_in_batches(G):
    rng = np.random.default_rng(3)
    probs = [(spread(rng, 2 + i % 3, 80, 20 + 60 * (i % 5)), 80, 2 + 6 * (i % 6)) for i in range(9)]
    ctx = G.Context(0)
    ctx.set_option(G.GD_OPT_GRID_LANES, 16)
    for rep in range(3):
        outs = ctx.dbscan_batched([(torch.from_numpy(x.astype(np.float32)).cuda(), e, m) for x, e, m in probs])
        for i, ((lab, core), (x, e, m)) in enumerate(zip(outs, probs)):
            want = oracle.dbscan(x, e, m)
            assert np.array_equal(core.cpu().numpy(), want[1]), f"call {rep} instance {i}"
            assert np.array_equal(lab.cpu().numpy(), want[0]), f"call {rep} instance {i}"
    ctx.close()
