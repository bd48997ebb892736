"""The two forms of the corridor network (rows, and CSR with arc records) at
the edges of what a row takes: 15 arcs in a vertex's own row, 16 more per
overflow row, 63 arcs at most, weights up to 32,767, and rows that fit the
arc memory.  Everything is compared with the oracle; the outputs are unique,
so the bar is bit-exact."""
import numpy as np
import pytest

import gen
import oracle
from tests.helpers import csr_from_edges

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.close()


def _band(n, h, wmax, seed):
    """Edges i .. i+1, ..., i+h (one more for even i): interior degrees 2h to
    2h+2, edge weights up to wmax, the largest one present."""
    rng = np.random.default_rng(seed)
    edges = [(i, j) for i in range(n) for j in range(i + 1, min(n, i + h + 1 + (i % 2 == 0)))]
    w = rng.integers(max(1, wmax // 2), wmax + 1, len(edges))
    w[len(edges) // 2] = wmax
    return csr_from_edges(n, edges, w.tolist())


def _check(fr, ctx, g, part, p, static=False):
    import torch

    print(f"rows n={g.n} maxdeg={np.diff(g.xadj).max()} maxw={g.adjwgt.max()} {p}", flush=True)
    o = oracle.refine_pair(g, part, 2, 0, 1, p, want_side=False)
    dg = fr.DeviceGraph.from_host(g)
    d = torch.as_tensor(part.copy()).cuda()
    prm = fr.params(**{k: v for k, v in p.items() if k in dict(fr.FrParams._fields_)})
    if static:
        res, tr = fr.flow_refine_pair_static(ctx, dg, d, 2, 0, 1, prm)
    else:
        res, tr, _ = fr.flow_refine_pair(ctx, dg, d, 2, 0, 1, prm)
    assert tr == o.trace
    assert res["cut_after"] == o.result["cut_after"]
    assert np.array_equal(d.cpu().numpy(), o.part)


def _split(g, seed, frac=0.05):
    part = (np.arange(g.n) >= g.n // 2).astype(np.int32)
    gen.pair_swap_noise(g, part, frac, seed)
    return part


BASE = dict(area_mode=0, depth=0, alpha=8, alpha_max=8, adaptive=1, max_iters=8, eps_ppm=50000)


@pytest.mark.parametrize("terminals,mb_reps", [(0, 0), (1, 0), (0, 4)])
@pytest.mark.parametrize("h", [1, 6, 7, 8, 15, 16, 30, 31, 32, 40])
def test_degrees(gpu_lib, ctx, h, terminals, mb_reps):
    g = _band(400 + h, h, 9, h)
    p = dict(BASE, terminals=terminals, mb_reps=mb_reps, mb_seed=3)
    _check(gpu_lib, ctx, g, _split(g, h), p)


@pytest.mark.parametrize("wmax", [1, 32767, 32768, 100000])
def test_weights(gpu_lib, ctx, wmax):
    g = _band(500, 5, wmax, 11)
    for terminals in (0, 1):
        _check(gpu_lib, ctx, g, _split(g, 4), dict(BASE, terminals=terminals))


@pytest.mark.parametrize("eps_ppm", [20000, 400000])
def test_static_arc_memory(gpu_lib, ctx, eps_ppm):
    """A grid's four arc records per vertex are half a row: small corridors
    fit as rows, one of nearly all vertices does not."""
    g = gen.grid2d(48, 48)
    part = (np.arange(g.n) % 48 >= 24).astype(np.int32)
    gen.pair_swap_noise(g, part, 0.1, 3)
    _check(gpu_lib, ctx, g, part, dict(BASE, eps_ppm=eps_ppm), static=True)


@pytest.mark.parametrize("threads,n", [(256, 3000), (512, 3000), (1024, 30000)])
def test_list_widths(gpu_lib, threads, n):
    """Frontiers of every width (8, 4 and 2 lanes per row) and lists longer
    than their LDS part, at each workgroup size."""
    g = gen.rgg(n, 3, 12.0, seed=5, wlo=1, whi=3)
    part = gen.rcb(g, 2)
    gen.global_noise(g, part, 0.2, 5)
    c = gpu_lib.Context()
    c.set_tuning(block_threads=threads)
    try:
        _check(gpu_lib, c, g, part, dict(BASE, alpha=16, alpha_max=16, eps_ppm=30000))
    finally:
        c.close()
