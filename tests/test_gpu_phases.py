"""Phase times of the neighbour lists, however they are built: counting and
filling each have their own, over all tree levels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    import paper_2210_07580_amd as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return G


# walks per grid (one dimension; ordered lists in three), levels (two, three and
# seven, in both orders), node lists (five and six, sparse)
@pytest.mark.parametrize("d,n,domain,eps", [(1, 5000, 20_000, 10), (2, 20_000, 3000, 40), (3, 20_000, 500, 100),
                                            (3, 20_000, 2000, 60), (5, 20_000, 1000, 150), (6, 20_000, 1000, 200),
                                            (7, 20_000, 60, 80)])
def test_counting_and_filling_are_timed_apart(G, d, n, domain, eps):
    x = np.random.default_rng(d).integers(0, domain, size=(n, d)).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    ctx = G.Context(0)
    assert sum(ctx.phase_times().values()) == 0
    ctx.set_option(G.GD_OPT_TIMING, 1)
    for _ in range(2):
        ctx.dbscan(t, eps, 5)
        ph = ctx.phase_times()
        for phase in ("minmax", "keys", "radix_sort", "cells", "grid_tree", "nei_count", "nei_fill", "core_mark",
                      "merge", "labels", "output"):
            assert 0 < ph[phase] < 1000, (phase, ph)
    ctx.set_option(G.GD_OPT_TIMING, 0)
    ctx.dbscan(t, eps, 5)
    assert sum(ctx.phase_times().values()) == 0
    ctx.close()
