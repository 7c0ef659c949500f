"""Split streams with a queue too small for their tasks: what does not fit is
streamed by the wave that asked, the slots left over are marked, and the
results are the oracle's."""
import numpy as np
import pytest

import oracle
from test_gpu_split import lumps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    import paper_2210_07580_amd as G
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return G


# no slot, one, an odd few (requests end short of them), about half of what is asked for
@pytest.mark.parametrize("slots", [0, 1, 7, 30])
@pytest.mark.parametrize("d", [1, 2, 3, 7])
@pytest.mark.parametrize("minpts,eps", [(3, 1000), (700, 1000), (700, 30_000)])
def test_full_queue(G, d, slots, minpts, eps):
    print(f"case d={d} slots={slots} minpts={minpts} eps={eps}", flush=True)
    x = lumps(d, d, (4097, 2048, 6500), eps, 6 if d == 1 else 10)
    want = oracle.dbscan(x, eps, minpts)
    t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()
    for options in ([], [(G.GD_OPT_STATS, 1)], [(G.GD_OPT_GRAPH, 2)]):
        ctx = G.Context(0)
        ctx.debug_limits(split_slots=slots)
        for k, v in options:
            ctx.set_option(k, v)
        for call in range(3):
            lab, core = ctx.dbscan(t, eps, minpts)
            assert np.array_equal(core.cpu().numpy(), want[1]), f"{options} call {call}"
            assert np.array_equal(lab.cpu().numpy(), want[0]), f"{options} call {call}"
        assert ctx.stats()["n"] >= 256 * ctx.stats()["grids"]
        ctx.close()


def test_limits_need_a_context(G):
    assert G.load_library().gd_debug_limits(None, 0, -1) == G.GD_EINVAL
