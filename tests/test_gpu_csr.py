"""The CSR form of the corridor network on the paths where most networks are
rows: rounds in slices of one microsecond whose solves continue in later
launches, rounds that mix both forms, the cut options on the launch chains,
captured and timed sweeps, and corridors beyond the LDS bitmaps.  An edge
above 32,767 or a vertex of more than 63 arcs in its corridor gives an entry
the CSR form.  Outputs are unique, so the bar is bit-exact with the oracle."""
import numpy as np
import pytest

import gen
import oracle
from tests.helpers import csr_from_edges, edges_of
from tests.test_gpu_parity import RESULT_KEYS, _batch_case
from tests.test_gpu_sliced import _batch_vs_oracle, _prm

pytestmark = pytest.mark.gpu

HEAVY = 40000
BASE = dict(area_mode=0, depth=0, alpha=16, alpha_max=16, adaptive=1, max_iters=16, eps_ppm=30000)


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.close()


@pytest.fixture(scope="module")
def sliced(gpu_lib):
    c = gpu_lib.Context()
    c.set_tuning(slice_us=1)
    yield c
    c.close()


def _heavy(g, part, blocks, share=40):
    """Weight HEAVY for one in `share` of the edges inside the given blocks,
    the same in both directions.  (A whole corridor's capacity stays below
    2^31: at most 50,000 heavy arcs.)"""
    u = np.repeat(np.arange(g.n, dtype=np.int64), np.diff(g.xadj))
    v = g.adjncy.astype(np.int64)
    h = (np.minimum(u, v) * 2654435761 + np.maximum(u, v) * 40503) % 1000003
    at = (h % share == 0) & (part[u] == part[v]) & np.isin(part[u], blocks)
    assert 0 < at.sum() < 50000
    g.adjwgt[at] = HEAVY
    return g


def _largest_class(g, part, k):
    edges, colour = oracle.quotient_colouring(g, part, k)
    cls = int(np.argmax(np.bincount(colour)))
    return [tuple(e) for e, c in zip(edges.tolist(), colour.tolist()) if c == cls]


def _case(seed, n, k, dim, forms):
    g, part = _batch_case(seed, n, k, dim=dim, deg=8.0 if dim == 2 else 12.0)
    pairs = _largest_class(g, part, k)
    csr = {"csr": pairs, "both": pairs[::2]}[forms]
    return _heavy(g, part, [b for p in csr for b in p]), part, pairs


@pytest.mark.parametrize("forms", ["csr", "both"])
@pytest.mark.parametrize("seed,n,k,dim", [(61, 1 << 15, 8, 2), (62, 1 << 15, 16, 3)])
def test_sliced_rounds(gpu_lib, sliced, seed, n, k, dim, forms):
    g, part, pairs = _case(seed, n, k, dim, forms)
    _, st = _batch_vs_oracle(gpu_lib, sliced, g, part, k, pairs, BASE)
    assert st["slices"] > 0


OPTIONS = [dict(cut_side=1), dict(cut_side=2), dict(terminals=1), dict(terminals=1, cut_side=2),
           dict(fm_limit=20, fm_seed=5), dict(mb_reps=4, mb_seed=3),
           dict(mb_reps=4, mb_seed=3, terminals=1)]


@pytest.mark.parametrize("forms", ["csr", "both"])
@pytest.mark.parametrize("opt", OPTIONS, ids=[",".join(f"{k}{v}" for k, v in o.items())
                                              for o in OPTIONS])
def test_options(gpu_lib, ctx, sliced, opt, forms):
    g, part, pairs = _case(63, 12000, 8, 2, forms)
    for c in (ctx, sliced):
        _batch_vs_oracle(gpu_lib, c, g, part, 8, pairs, dict(BASE, **opt))


def test_hubs(gpu_lib, sliced):
    """One vertex of 80 arcs in every other block: the misfit is the degree."""
    g, part = _batch_case(64, 1 << 14, 8)
    pairs = _largest_class(g, part, 8)
    edges = {(u, v): w for u, v, w in edges_of(g)}
    rng = np.random.default_rng(64)
    for a, b in pairs[::2]:
        # next to the cut, so that every corridor holds it
        hub = next(u for u, v, _ in edges_of(g) if (part[u], part[v]) in ((a, b), (b, a)))
        mine = np.nonzero(part == part[hub])[0]
        for v in rng.choice(mine, 80, replace=False):
            if v != hub:
                edges[min(hub, int(v)), max(hub, int(v))] = 3
    h = csr_from_edges(g.n, list(edges), list(edges.values()), g.vwgt)
    assert np.diff(h.xadj).max() > 63
    _batch_vs_oracle(gpu_lib, sliced, h, part, 8, pairs, BASE)


@pytest.mark.parametrize("timing", [False, True])
@pytest.mark.parametrize("active", [0, 1])
def test_sweeps(gpu_lib, sliced, timing, active):
    """Captured (not sliced) and launched round by round (sliced)."""
    import torch

    g, part = _batch_case(65 + active, 1 << 14, 16)
    g = _heavy(g, part, list(range(0, 16, 3)))
    p = dict(BASE, active_blocks=active, fm_limit=20 * active, fm_seed=3)
    rc, tc, stats, opart = oracle.sweep(g, part, 16, p, max_sweeps=4)
    assert rc == 0
    sliced.set_timing(timing)
    try:
        d = torch.as_tensor(part.copy()).cuda()
        tc_gpu, st_gpu = gpu_lib.flow_refine_sweep(sliced, gpu_lib.DeviceGraph.from_host(g), d, 16,
                                                   _prm(gpu_lib, p), 4)
    finally:
        sliced.set_timing(False)
    assert tc_gpu == tc
    assert st_gpu.tolist() == stats.tolist()
    assert np.array_equal(d.cpu().numpy(), opart)


@pytest.mark.parametrize("terminals,cut_side", [(0, 1), (1, 0)])
def test_corridor_beyond_lds_bitmaps(gpu_lib, ctx, terminals, cut_side):
    """More than 131,072 corridor vertices: the searches' marks and the labels
    of the CSR form live in device memory."""
    import torch

    w = gen.config("C2", n_override=1 << 19)
    g = _heavy(w.graph, w.part, [0, 1], share=500)
    p = {k: w.params[k] for k in ("area_mode", "depth", "alpha", "alpha_max", "eps_ppm")}
    p.update(adaptive=0, max_iters=1, terminals=terminals, cut_side=cut_side)
    o = oracle.refine_pair(g, w.part, 2, 0, 1, p, want_side=True)
    assert o.result["region_vertices"] > 131072
    d = torch.as_tensor(w.part.copy()).cuda()
    res, trace, side = gpu_lib.flow_refine_pair(ctx, gpu_lib.DeviceGraph.from_host(g), d, 2, 0, 1,
                                                _prm(gpu_lib, p), want_side=True)
    for key in RESULT_KEYS:
        assert res[key] == o.result[key], key
    assert trace == o.trace
    assert np.array_equal(side, o.side)
    assert np.array_equal(d.cpu().numpy(), o.part)
