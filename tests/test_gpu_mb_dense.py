"""Most balanced cuts on row networks of more than 16 arcs per vertex, where
the arc lists of an entry (its one-way arcs, then the quotient graph's, beyond
LDS) take more words than the entry's network rows take records.

The graph is a thick path: layers of w vertices, each joined to every vertex
of the next.  A flow from end to end saturates all arcs, so every inner vertex
is a class of its own and every arc of the corridor is one-way: the two lists
of w^2 words per pair of layers come close to the corridor's arc count."""
import numpy as np
import pytest

import gen
import oracle
from tests.helpers import csr_from_edges

pytestmark = pytest.mark.gpu


def _thick_path(layers, w):
    edges = [(w * i + a, w * i + w + b) for i in range(layers - 1) for a in range(w)
             for b in range(w)]
    return csr_from_edges(layers * w, edges)


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.close()


def _check(fr, ctx, g, part, k, pairs, p):
    import torch

    print(f"dense mb n={g.n} maxdeg={np.diff(g.xadj).max()} k={k} {p}", flush=True)
    rc, ores, otr, opart = oracle.refine_batch(g, part, k, pairs, p)
    assert rc == 0
    d = torch.as_tensor(part.copy()).cuda()
    res, tr = fr.flow_refine_batch(ctx, fr.DeviceGraph.from_host(g), d, k, pairs, fr.params(**p))
    for i in range(len(pairs)):
        assert tr[i] == otr[i], pairs[i]
        assert res[i]["cut_after"] == ores[i]["cut_after"]
    assert np.array_equal(d.cpu().numpy(), opart)
    return fr.stats_dict(ctx)


P = dict(area_mode=0, depth=0, alpha=16, alpha_max=16, adaptive=1, max_iters=6, mb_reps=4,
         mb_seed=5)


@pytest.mark.parametrize("layers,w,eps_ppm", [(30, 20, 60000), (60, 20, 55000), (40, 31, 60000),
                                              (41, 9, 60000), (40, 8, 30000)])
def test_thick_path(gpu_lib, ctx, layers, w, eps_ppm):
    g = _thick_path(layers, w)
    part = (np.arange(g.n) >= w * (layers // 2)).astype(np.int32)
    st = _check(gpu_lib, ctx, g, part, 2, [(0, 1)], dict(P, eps_ppm=eps_ppm))
    assert st["slots"] == 5 and st["mb_free"] > 0


@pytest.mark.parametrize("speculate", [True, False])
def test_round_of_thick_paths(gpu_lib, ctx, speculate):
    """Three pairs, with their speculative chains and without: neighbouring
    entries of the arena are slots of one pair, or different pairs."""
    layers, w = 30, 20
    one = _thick_path(layers, w)
    edges = [(u + c * one.n, int(v) + c * one.n) for c in range(3) for u in range(one.n)
             for v in one.adjncy[one.xadj[u]:one.xadj[u + 1]] if v > u]
    g = csr_from_edges(3 * one.n, edges)
    part = (np.arange(g.n) // (w * (layers // 2))).astype(np.int32)
    ctx.set_speculation(speculate)
    try:
        st = _check(gpu_lib, ctx, g, part, 6, [(0, 1), (2, 3), (4, 5)], dict(P, eps_ppm=55000))
    finally:
        ctx.set_speculation(True)
    assert st["mb_free"] > 0
