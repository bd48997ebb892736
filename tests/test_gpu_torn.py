"""Input whose checks are switched off: an arc without its reverse inside a
corridor is still found when the network is built, in both of its forms, and
the call reports FR_E_INVALID_GRAPH with the partition untouched; repeated
edges and self loops are harmless."""
import numpy as np
import pytest

import oracle
from gen import Graph
from tests.helpers import csr_from_edges

pytestmark = pytest.mark.gpu

SIDE = 24
PRM = dict(area_mode=1, depth=6, alpha=1, alpha_max=1, adaptive=0, max_iters=1, eps_ppm=100000)


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    c.set_validation(False)
    yield c
    c.close()


def _grid():
    edges = [(SIDE * y + x, SIDE * y + x + 1) for y in range(SIDE) for x in range(SIDE - 1)]
    edges += [(SIDE * y + x, SIDE * y + SIDE + x) for y in range(SIDE - 1) for x in range(SIDE)]
    w = np.random.default_rng(5).integers(1, 6, len(edges)).tolist()
    return edges, w, (np.arange(SIDE * SIDE) % SIDE >= SIDE // 2).astype(np.int32)


def _run(fr, ctx, g, part, **kw):
    import torch

    d = torch.as_tensor(part.copy()).cuda()
    dg, prm = fr.DeviceGraph.from_host(g), fr.params(**dict(PRM, **kw))
    print(f"torn n={g.n} arcs={len(g.adjncy)} {kw}", flush=True)
    res, tr, _ = fr.flow_refine_pair(ctx, dg, d, 2, 0, 1, prm)
    return res, tr, d.cpu().numpy()


def _without(g, tail, head):
    """The graph without the one arc tail -> head."""
    e = int(g.xadj[tail]) + int(np.nonzero(g.adjncy[g.xadj[tail]:g.xadj[tail + 1]] == head)[0][0])
    xadj = g.xadj.copy()
    xadj[tail + 1:] -= 1
    return Graph(xadj, np.delete(g.adjncy, e), np.delete(g.adjwgt, e), g.vwgt.copy())


@pytest.mark.parametrize("form", ["rows", "csr"])
@pytest.mark.parametrize("mb_reps", [0, 2])
@pytest.mark.parametrize("upper", [False, True])
def test_missing_reverse_arc(gpu_lib, ctx, form, mb_reps, upper):
    """Either direction of an edge two columns from the cut, inside block 0."""
    edges, w, part = _grid()
    u = SIDE * 7 + SIDE // 2 - 3
    if form == "csr":
        w[edges.index((u, u + 1))] = 40000
    g = csr_from_edges(SIDE * SIDE, edges, w)
    bad = _without(g, *((u, u + 1) if upper else (u + 1, u)))
    with pytest.raises(gpu_lib.FlowRefineError) as e:
        _run(gpu_lib, ctx, bad, part, mb_reps=mb_reps)
    assert e.value.code == -1
    assert gpu_lib.stats_dict(ctx)["diag"] == 3
    # the whole graph refines on the same context
    o = oracle.refine_pair(g, part, 2, 0, 1, dict(PRM, mb_reps=mb_reps))
    res, tr, out = _run(gpu_lib, ctx, g, part, mb_reps=mb_reps)
    assert tr == o.trace and np.array_equal(out, o.part)


def test_repeated_edges_and_self_loops(gpu_lib, ctx):
    """Two edges of weights x and y between two vertices cut like one of x + y,
    and a self loop like none."""
    edges, w, part = _grid()
    g = csr_from_edges(SIDE * SIDE, edges, w)
    rng = np.random.default_rng(8)
    adj = [[] for _ in range(g.n)]
    for (u, v), x in zip(edges, w):
        parts = [x]
        if x > 1 and rng.random() < 0.3:
            parts = [1, x - 1]
        for y in parts:
            adj[u].append((v, y))
            adj[v].append((u, y))
    for u in rng.choice(g.n, 60, replace=False):
        adj[u].append((int(u), 3))
    for row in adj:
        row.sort()
    flat = [a for row in adj for a in row]
    h = Graph(np.cumsum([0] + [len(r) for r in adj]).astype(np.int32),
              np.asarray([v for v, _ in flat], dtype=np.int32),
              np.asarray([y for _, y in flat], dtype=np.int32), g.vwgt.copy())
    o = oracle.refine_pair(g, part, 2, 0, 1, PRM)
    res, _, out = _run(gpu_lib, ctx, h, part)
    assert res["flow_value"] == o.result["flow_value"]
    assert res["cut_after"] == o.result["cut_after"]
    assert np.array_equal(out, o.part)
