"""The corridor search at the edges of its forms: levels of one to several
vertices per lane group (narrow up to 256 vertices), more vertices per level
than have an entry in local memory (2,048), both sides cut inside a level,
degrees around a step of 16 arcs, and a graph whose bitmap of reached vertices
doesn't fit a CU.  Everything is compared with the oracle; corridors and
results are unique, so the bar is bit-exact."""
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


def _grid(rows, cols, seed):
    """rows x cols grid graph with weights in 1..5, split between the middle
    columns: a boundary of 2 * rows vertices."""
    rng = np.random.default_rng(seed)
    n = rows * cols
    at = np.arange(n).reshape(rows, cols)
    e = np.concatenate([np.stack([at[:, :-1].ravel(), at[:, 1:].ravel()]),
                        np.stack([at[:-1].ravel(), at[1:].ravel()])], axis=1)
    w = rng.integers(1, 6, e.shape[1])
    src, dst = np.concatenate([e[0], e[1]]), np.concatenate([e[1], e[0]])
    ww = np.concatenate([w, w])
    order = np.lexsort((dst, src))
    xadj = np.zeros(n + 1, dtype=np.int32)
    xadj[1:] = np.cumsum(np.bincount(src, minlength=n))
    g = type(csr_from_edges(2, [(0, 1)]))(xadj, dst[order].astype(np.int32),
                                          ww[order].astype(np.int32),
                                          rng.integers(1, 6, n).astype(np.int32))
    return g, (at % cols >= cols // 2).astype(np.int32).ravel()


def _check(fr, ctx, g, part, p):
    import torch

    print(f"corridor n={g.n} {p}", flush=True)
    o = oracle.refine_pair(g, part, 2, 0, 1, p, want_side=False)
    dg = fr.DeviceGraph.from_host(g)
    d = torch.as_tensor(part.copy()).cuda()
    prm = fr.params(**{k: v for k, v in p.items() if k in dict(fr.FrParams._fields_)})
    res, tr, _ = fr.flow_refine_pair(ctx, dg, d, 2, 0, 1, prm)
    assert tr == o.trace
    for key in ("region_vertices", "region_edges", "cut_after"):
        assert res[key] == o.result[key], key
    assert np.array_equal(d.cpu().numpy(), o.part)


DEPTH = dict(area_mode=1, alpha=1, alpha_max=1, adaptive=0, max_iters=1, eps_ppm=50000)
AREA = dict(area_mode=0, depth=0, alpha=4, alpha_max=4, adaptive=1, max_iters=4, eps_ppm=30000)


@pytest.mark.parametrize("rows", [1, 31, 63, 64, 65, 127, 128, 129, 255, 256, 257, 1023, 1024,
                                  1025, 2100])
def test_level_widths(gpu_lib, ctx, rows):
    g, part = _grid(rows, 40, rows)
    _check(gpu_lib, ctx, g, part, dict(DEPTH, depth=6))
    _check(gpu_lib, ctx, g, part, AREA)


@pytest.mark.parametrize("deg", [7, 8, 9, 15, 16, 17, 31, 33, 70])
def test_degrees(gpu_lib, ctx, deg):
    n = 4000
    edges = {(i, (i + d * d) % n) for i in range(n) for d in range(1, deg // 2 + 1)}
    if deg % 2:
        edges |= {(i, i + n // 2) for i in range(n // 2)}
    edges = sorted({(min(e), max(e)) for e in edges if e[0] != e[1]})
    g = csr_from_edges(n, edges)
    part = (np.arange(n) >= n // 2).astype(np.int32)
    gen.pair_swap_noise(g, part, 0.02, deg)
    _check(gpu_lib, ctx, g, part, AREA)
    _check(gpu_lib, ctx, g, part, dict(DEPTH, depth=1))


@pytest.mark.parametrize("rows,cols", [(150, 8000), (3000, 400)])
def test_graph_beyond_the_bitmap(gpu_lib, ctx, rows, cols):
    g, part = _grid(rows, cols, 7)
    _check(gpu_lib, ctx, g, part, dict(DEPTH, depth=4))
