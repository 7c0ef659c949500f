"""Calls on a device without memory to spare (gd_debug_limits): what fails
leaves the context and the last call's views as they were, and what the call
can do without is given up first."""
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


def check(ctx, x, eps, minpts):
    lab, core = ctx.dbscan(dev(x), eps, minpts)
    want = oracle.dbscan(x, eps, minpts)
    assert np.array_equal(core.cpu().numpy(), want[1])
    assert np.array_equal(lab.cpu().numpy(), want[0])


def uniform(seed, n, d, domain):
    return np.random.default_rng(seed).integers(0, domain, size=(n, d)).astype(np.int32)


@pytest.mark.parametrize("d", [2, 5])
def test_batch_table_that_does_not_fit(G, d):
    # a longer table than the context has fails; the call before it can still
    # be inspected and the next calls work
    x = uniform(d, 4000, d, 600)
    ctx, ref = G.Context(0), G.Context(0)
    ref.set_option(G.GD_OPT_NEIGHBOR_MODE, 1)
    check(ref, x, 90, 4)
    check(ctx, x, 90, 4)
    before = ctx.stats()
    ctx.debug_limits(device_bytes=0)
    few = [(dev(x[:50]), 90, 4)] * 40
    with pytest.raises(G.GDError) as e:
        ctx.dbscan_batched(few)
    assert e.value.status == G.GD_ENOMEM
    ctx.debug_limits()
    assert ctx.stats() == before
    for got, want in zip(ctx.debug_neighbors(), ref.debug_neighbors()):
        assert np.array_equal(got, want)
    check(ctx, x, 80, 5)
    lab, core = oracle.dbscan(x[:50], 90, 4)
    for got in ctx.dbscan_batched(few):
        assert np.array_equal(got[0].cpu().numpy(), lab) and np.array_equal(got[1].cpu().numpy(), core)
    ctx.close()
    ref.close()


def node_list_call(ctx, n=20_000):
    # six dimensions: the lists of the level above the families' own take megabytes
    check(ctx, uniform(6, n, 6, 1000), 200, 5)


def test_a_workspace_limit_gives_the_node_lists_back(G):
    ctx = G.Context(0)
    node_list_call(ctx)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.set_option(G.GD_OPT_WORKSPACE_LIMIT, 1 << 30)
    assert torch.cuda.mem_get_info()[0] >= free + (1 << 20)
    node_list_call(ctx)
    ctx.set_option(G.GD_OPT_WORKSPACE_LIMIT, 0)
    node_list_call(ctx)
    ctx.close()


def test_node_lists_make_room_for_a_later_call(G):
    # what a fresh context can do with so much memory, one that built node
    # lists before (smaller than the later call's own lists) can do too
    x = uniform(2, 400_000, 2, 30_000)

    def fits(limit, before):
        ctx = G.Context(0)
        if before:
            node_list_call(ctx, 4000)
        ctx.debug_limits(device_bytes=limit)
        try:
            check(ctx, x, 100, 4)
            return True
        except G.GDError as e:
            assert e.status == G.GD_ENOMEM
            return False
        finally:
            ctx.close()

    lo, hi = 1 << 20, 1 << 29
    assert not fits(lo, False) and fits(hi, False)
    while hi - lo > 1 << 16:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fits(mid, False) else (mid, hi)
    assert fits(hi, True)
