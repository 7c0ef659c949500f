"""Clustering calls that a user of this package makes, over the range it is
used in: single calls from a thousand to twenty million points in two to
seven dimensions, dense seed-spreader walks and sparse blobs, one- and
two-word grid identifiers, whole batches, the allocation-free entry and the
learned merge proposal.

Points are drawn on the GPU from the seed alone, with the recipes of the
seeded workloads of this repository (Gaussian blobs plus uniform noise; a
seed spreader that emits points in a ball, moves on and now and then jumps),
integer coordinates as float32, rows in random order.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2210_07580_amd as G

# Recipes (domain, blobs, spreader steps) of the seeded workloads.
BLOB2 = {"kind": "blobs", "domain": 10_000, "blobs": 10, "sigma_lo": 200.0, "sigma_hi": 200.0, "noise": 0.10}
BLOB5 = {"kind": "blobs", "domain": 1_000_000, "blobs": 100, "sigma_lo": 2_000.0, "sigma_hi": 20_000.0, "noise": 0.01}
WALK = {"kind": "walk", "domain": 100_000, "step": 50.0, "levels": 1, "noise": 1e-4}


def _sweep(d: int, n: int, levels: int) -> dict:
    """The parameter sweeps' data: about ten walks whatever n, steps of 50 d;
    levels 1: walks of similar density, 4: of varying density."""
    return {"kind": "walk", "domain": 100_000, "step": 50.0 * d, "levels": levels, "noise": 1e-4, "per_step": 100,
            "restart": min(1.0, 1000.0 / n)}


def listed() -> list[dict]:
    sweep_n = 2_000_000
    return [
        # an interactive call: latency, launches and read-backs are all there is
        {"name": "blobs_2d_1k", "call": "single", "n": 1_000, "d": 2, "eps": 100, "minpts": 10, **BLOB2},
        # the small 2-D set of the test suite and the smoke check
        {"name": "blobs_2d_10k", "call": "single", "n": 10_000, "d": 2, "eps": 100, "minpts": 10, **BLOB2},
        # a serving loop that may not allocate: the entry with the fixed workspace, an odd size
        {"name": "noalloc_3d_300k", "call": "noalloc", "n": 300_007, "d": 3, "eps": 200, "minpts": 100, **WALK,
         "per_step": 100, "restart": 0.001},
        # a wide radius on 2-D data: a few hundred grids of up to 3e5 points
        {"name": "walk_2d_2m_eps5000", "call": "single", "n": sweep_n, "d": 2, "eps": 5_000, "minpts": 100,
         **_sweep(2, sweep_n, 1)},
        # the ordinary 3-D call of the benchmark plan
        {"name": "walk_3d_2m", "call": "single", "n": 2_000_000, "d": 3, "eps": 200, "minpts": 100, **WALK,
         "per_step": 100, "restart": 0.001},
        # the headline workload of bench.py
        {"name": "walk_3d_10m", "call": "single", "n": 10_000_000, "d": 3, "eps": 200, "minpts": 100, **WALK,
         "per_step": 100, "restart": 0.001},
        # the densest single call of the benchmark plan, 33-bit identifiers
        {"name": "walk_3d_20m", "call": "single", "n": 20_000_000, "d": 3, "eps": 150, "minpts": 50, **WALK,
         "per_step": 300, "restart": 0.001},
        # millions of tiny grids: neighbour lists of billions of entries
        {"name": "blobs_5d_10m", "call": "single", "n": 10_000_000, "d": 5, "eps": 5_000, "minpts": 20, **BLOB5},
        # a middle point of the parameter sweeps in seven dimensions, varying density
        {"name": "walk_7d_2m", "call": "single", "n": sweep_n, "d": 7, "eps": 2_000, "minpts": 100,
         **_sweep(7, sweep_n, 4)},
        # a small radius in seven dimensions: 70-bit identifiers (two words), an odd size
        {"name": "walk_7d_1m_eps500", "call": "single", "n": 1_000_003, "d": 7, "eps": 500, "minpts": 25,
         **_sweep(7, 1_000_003, 1)},
        # many data sets of different sizes at once, replayed from the second call on
        {"name": "batch_256", "call": "batch", "count": 256, "n_lo": 1_000, "n_hi": 1_000_000, "sizes": 20221017,
         **BLOB2},
        # core sets of thousands of points with the trained merge proposal switched on
        {"name": "learned_3d_2m", "call": "learned", "n": sweep_n, "d": 3, "eps": 2_000, "minpts": 100,
         **_sweep(3, sweep_n, 1)},
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random) -> dict:
    what = rng.choice(("blobs", "walk", "sweep", "sweep", "blobs5", "batch", "noalloc", "learned"))
    if what == "blobs":
        return {"call": "single", "n": _log_int(rng, 1_000, 2_000_000), "d": rng.randint(2, 3),
                "eps": rng.randint(50, 300), "minpts": rng.randint(5, 50), **BLOB2}
    if what == "walk":
        return {"call": "single", "n": _log_int(rng, 100_000, 20_000_000), "d": 3, "eps": rng.randint(100, 300),
                "minpts": rng.randint(20, 100), **WALK, "per_step": rng.randint(100, 300), "restart": 0.001}
    if what == "sweep":
        d = rng.choice((2, 3, 5, 7))
        n = _log_int(rng, 100_000, 10_000_000 if d <= 3 else 4_000_000 if d == 5 else 2_000_000)
        return {"call": "single", "n": n, "d": d, "eps": rng.randint(500, 5_000), "minpts": rng.randint(10, 100),
                **_sweep(d, n, rng.choice((1, 4)))}
    if what == "blobs5":
        return {"call": "single", "n": _log_int(rng, 100_000, 5_000_000), "d": 5, "eps": rng.randint(4_000, 5_000),
                "minpts": rng.randint(10, 50), **BLOB5}
    if what == "batch":
        return {"call": "batch", "count": _log_int(rng, 4, 256), "n_lo": 1_000,
                "n_hi": _log_int(rng, 10_000, 1_000_000), "sizes": rng.randrange(1 << 30), **BLOB2}
    if what == "noalloc":
        return {"call": "noalloc", "n": _log_int(rng, 1_000, 500_000), "d": 3, "eps": rng.randint(150, 300),
                "minpts": rng.randint(20, 100), **WALK, "per_step": 100, "restart": 0.001}
    n = _log_int(rng, 500_000, 5_000_000)
    return {"call": "learned", "n": n, "d": 3, "eps": rng.randint(1_000, 3_000), "minpts": rng.randint(10, 100),
            **_sweep(3, n, rng.choice((1, 4)))}


def _instances(case: dict) -> list[tuple[int, int, int, int]]:
    """(n, d, eps, minpts) of every data set of the call; sizes and
    parameters belong to the case, only the points come from the seed."""
    if case["call"] != "batch":
        return [(case["n"], case["d"], case["eps"], case["minpts"])]
    rng = random.Random(case["sizes"])
    return [(_log_int(rng, case["n_lo"], case["n_hi"]), rng.randint(2, 3), rng.randint(50, 300), rng.randint(5, 50))
            for _ in range(case["count"])]


def _blobs(case: dict, sizes: list[int], d: int, g: torch.Generator, dev) -> torch.Tensor:
    """Rows of all data sets after each other, each with its own blobs."""
    n, k, L = sum(sizes), case["blobs"], float(case["domain"])
    centres = torch.rand(len(sizes) * k, d, generator=g, device=dev) * L
    sig = torch.rand(len(sizes) * k, d, generator=g, device=dev)
    sig = case["sigma_lo"] * (case["sigma_hi"] / case["sigma_lo"]) ** sig
    first = torch.repeat_interleave(torch.arange(len(sizes), device=dev) * k, torch.tensor(sizes, device=dev),
                                    output_size=n)
    owner = first + torch.randint(k, (n,), generator=g, device=dev)
    x = torch.randn(n, d, generator=g, device=dev).mul_(sig[owner]).add_(centres[owner])
    noise = torch.rand(n, 1, generator=g, device=dev) < case["noise"]
    return torch.where(noise, torch.rand(n, d, generator=g, device=dev) * L, x)


def _walk(case: dict, n: int, d: int, g: torch.Generator, dev) -> torch.Tensor:
    """Seed spreader: per_step points in a ball of radius 100 around each
    location of a random walk that is reflected at the walls and jumps with
    probability restart; levels > 1 scales a walk's ball and step by 2**k."""
    L, per = float(case["domain"]), case["per_step"]
    steps = -(-n // per)
    f64 = {"generator": g, "device": dev, "dtype": torch.float64}
    jump = torch.rand(steps, **f64) < case["restart"]
    jump[0] = True
    walk = torch.cumsum(jump, 0) - 1
    count = int(walk[-1]) + 1
    start = torch.rand(count, d, **f64) * L
    scale = torch.exp2(torch.randint(case["levels"], (count,), generator=g, device=dev).double())[walk]
    move = torch.randn(steps, d, **f64)
    move = move / move.norm(dim=1, keepdim=True) * (case["step"] * scale)[:, None]
    path = torch.cumsum(move, 0) - move
    path = path - path[jump][walk] + start[walk]
    path = L - (path.remainder(2.0 * L) - L).abs()  # a free path folded at the walls
    order = torch.randperm(n, generator=g, device=dev)
    owner = order // per
    x = torch.randn(n, d, generator=g, device=dev)
    r = 100.0 * torch.rand(n, generator=g, device=dev) ** (1.0 / d) * scale[owner].float()
    x.mul_((r / x.norm(dim=1))[:, None]).add_(path[owner].float())
    noise = order >= n - int(round(case["noise"] * n))
    return torch.where(noise[:, None], torch.rand(n, d, generator=g, device=dev) * L, x)


def _points(case: dict, seed: int) -> list[torch.Tensor]:
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    inst = _instances(case)
    d = max(q[1] for q in inst)
    sizes = [q[0] for q in inst]
    x = _blobs(case, sizes, d, g, dev) if case["kind"] == "blobs" else _walk(case, sizes[0], d, g, dev)
    x = x.round_().clamp_(0.0, float(case["domain"]))
    return [p[:, :q[1]].contiguous() for p, q in zip(x.split(sizes), inst)]


def prepare(case: dict, seed: int) -> dict:
    inst, points = _instances(case), _points(case, seed)
    ctx = G.Context(0)
    state = {"call": case["call"], "ctx": ctx, "problems": [(p, q[2], q[3]) for p, q in zip(points, inst)]}
    if case["call"] == "learned":
        from paper_2210_07580_amd import proposal
        ctx.set_proposal(proposal.load_blob())
    if case["call"] in ("noalloc", "batch"):
        # the program's own output arrays; a batch writes one stretch per data set
        sizes = [q[0] for q in inst]
        state["labels"] = torch.empty(sum(sizes), dtype=torch.int32, device="cuda:0")
        state["core"] = torch.empty(sum(sizes), dtype=torch.uint8, device="cuda:0")
        state["outs"] = list(zip(state["labels"].split(sizes), state["core"].split(sizes)))
    return state


def run(state: dict):
    ctx = state["ctx"]
    if state["call"] == "batch":
        ctx.dbscan_batched(state["problems"], outs=state["outs"])
        return state["labels"], state["core"]
    points, eps, minpts = state["problems"][0]
    if state["call"] == "noalloc":
        return ctx.dbscan_noalloc(points, eps, minpts, state["labels"], state["core"])
    return ctx.dbscan(points, eps, minpts)


def work(case: dict) -> dict:
    """Coordinates read once, a 4-byte label and a flag byte written per
    point; the arithmetic of each coordinate's grid identifier (subtract,
    multiply, floor, check)."""
    inst = _instances(case)
    return {"bytes": sum(n * (4 * d + 5) for n, d, _, _ in inst), "flops": sum(4 * n * d for n, d, _, _ in inst)}


def exact(case: dict, seed: int):
    """DBSCAN from all pair distances in 64 bits (small single calls only):
    a cluster's label is its smallest core index, a border point takes that
    of its lowest-index core neighbour, noise is -1."""
    if case["call"] != "single" or case["n"] > 12_000:
        return None
    n, eps2 = case["n"], float(case["eps"]) ** 2
    x = _points(case, seed)[0].double()
    rows, cols = [], []
    for i in range(0, n, 1_000):
        near = sum((x[i:i + 1_000, None, j] - x[None, :, j]) ** 2 for j in range(case["d"])) <= eps2
        r, c = near.nonzero(as_tuple=True)
        rows.append(r + i)
        cols.append(c)
    rows, cols = torch.cat(rows), torch.cat(cols)
    core = torch.bincount(rows, minlength=n) >= case["minpts"]
    a, b = rows[core[rows] & core[cols]], cols[core[rows] & core[cols]]
    label = torch.arange(n, device=x.device)
    while True:
        low = label.scatter_reduce(0, a, label[b], "amin")
        low = low[low]
        if torch.equal(low, label):
            break
        label = low
    to_core = core[cols]
    first = torch.full((n,), n, device=x.device).scatter_reduce(0, rows[to_core], cols[to_core], "amin")
    border = ~core & (first < n)
    label = torch.where(core, label, torch.where(border, label[first.clamp(max=n - 1)], -torch.ones_like(label)))
    return label.int(), core.to(torch.uint8)
