"""Performance cases of the flow refinement library.

Each case is one call of a public entry point on seeded synthetic input: the
graphs are those of the repository's own workloads (unit grids, 2D and 3D
random geometric graphs, unit or 1..10 edge weights, recursive coordinate
bisection plus boundary noise), at the sizes of its configurations and at odd
ones between them.  Graphs are built on the GPU, so preparing a case is quick.

listed() / draw(rng)   the cases, and one more of the same ranges
prepare(case, seed)    inputs and the handle a program holds before the call
run(state)             one pass through the entry point
work(case)             bytes and operations that a pass cannot do without
exact(case, seed)      float outputs in 64 bits (the network's gradient)
"""
import math

import numpy as np
import torch

import paper_1012_0006_amd as fr

RESULT = [f for f, _ in fr.FrResult._fields_]
SOLVE = [f for f, _ in fr.FrSolve._fields_]
SIDE_BITS = 20  # points are drawn on a lattice of 2^20 cells per axis


# ------------------------------------------------------------------ cases ---

def _graph(n, dim, deg, whi, k, noise):
    return dict(graph="rgg", n=n, dim=dim, deg=deg, whi=whi, k=k, noise=noise)


def listed():
    return [
        # The smallest call: one corridor of fixed depth on a 128 x 128 grid, one solve.  An
        # application that refines many small pairs pays mostly launches and waits.
        dict(name="grid-depth-pair", call="pair", graph="grid", n=128 * 128, k=2, noise=0.05,
             area_mode=1, depth=8, alpha=1, alpha_max=1, adaptive=0, max_iters=1),
        # A partitioner without GPU buffers: the graph and partition lie in host memory, as on
        # the coarse levels of a multilevel scheme.
        dict(_graph(5003, 2, 8.0, 10, 2, 0.02), name="host-pair", call="pair_host"),
        # The entry point that allocates nothing, for serving loops and captured code.
        dict(_graph(60013, 2, 8.0, 10, 4, 0.02), name="static-pair", call="pair_static"),
        # One large pair refined adaptively: the finest level of a bisection.
        dict(_graph(1 << 18, 2, 8.0, 10, 2, 0.02), name="rgg2d-pair", call="pair"),
        # A matching round over few large blocks of a 3D mesh-like graph: wide corridors.
        dict(_graph(1 << 20, 3, 12.0, 1, 16, 0.02), name="rgg3d-round", call="batch"),
        # A matching round over many blocks of a 2D graph: the inner step of a k-way scheduler.
        dict(_graph(1 << 22, 2, 6.0, 1, 64, 0.01), name="rgg2d-round", call="batch"),
        # A round with the quality options: local search first, then contracted terminals and
        # the most balanced minimum cut; an odd size.
        dict(_graph(1000003, 2, 8.0, 10, 16, 0.02), name="quality-round", call="batch",
             fm_limit=100, mb_reps=16, terminals=1),
        # Multi-try local search after a round's pairwise improvement.
        dict(_graph(1 << 17, 3, 12.0, 1, 8, 0.02), name="multitry-round", call="batch",
             mt_alpha=10),
        # Refinement of a whole partition until no pair improves.
        dict(_graph((1 << 20) + 7, 2, 6.0, 1, 16, 0.01), name="sweep", call="sweep",
             max_sweeps=32),
        # The same with active blocks, local search and balanced cuts; k no power of two.
        dict(_graph(300007, 2, 8.0, 10, 24, 0.02), name="active-sweep", call="sweep",
             max_sweeps=32, fm_limit=100, mb_reps=16, active_blocks=1),
        # One pass over all pairs of a large graph from the learned start factors.
        dict(_graph(1 << 22, 2, 8.0, 10, 64, 0.02), name="learned-sweep", call="sweep",
             max_sweeps=1, use_mlp=1),
        # Training the start-factor network: loss and gradient over a set of labelled pairs.
        dict(name="mlp-gradient", call="mlp", n=16384, costs=1),
    ]


def _size(rng, lo, hi):
    """Log-uniform size in [lo, hi], odd two times in three."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(hi, n | 1) if rng.random() < 0.67 else n


def draw(rng):
    call = rng.choice(("pair", "pair", "pair_host", "pair_static", "batch", "batch", "batch",
                       "sweep", "sweep", "mlp"))
    if call == "mlp":
        return dict(call="mlp", n=_size(rng, 64, 16384), costs=rng.randrange(2))
    dim = rng.choice((2, 2, 3))
    whi = rng.choice((1, 10))
    noise = rng.choice((0.01, 0.02, 0.05))
    if call in ("pair", "pair_host", "pair_static"):
        k = rng.choice((2, 2, 3, 4, 8))
        hi = {"pair": 1 << 18, "pair_host": 1 << 16, "pair_static": 60013}[call]
        if call == "pair" and rng.random() < 0.25:
            side = rng.randrange(24, 161)
            return dict(call="pair", graph="grid", n=side * side, k=2, noise=noise, area_mode=1,
                        depth=rng.randrange(2, 13), alpha=1, alpha_max=1, adaptive=0, max_iters=1)
        n = _size(rng, 1024, hi)
        n = min(n, 1 << 16) if dim == 3 else n
    else:
        k = rng.randrange(4, 65)
        hi = {("batch", 2): 1 << 21, ("batch", 3): 1 << 19,
              ("sweep", 2): 1 << 19, ("sweep", 3): 1 << 16}[call, dim]
        n = _size(rng, 512 * k, max(hi, 1024 * k))
    deg = {2: rng.choice((6.0, 8.0)), 3: 12.0}[dim]
    case = dict(_graph(n, dim, deg, whi, k, noise), call=call)
    if call == "sweep":
        case.update(max_sweeps=rng.choice((1, 4, 32)), use_mlp=rng.randrange(2),
                    active_blocks=rng.randrange(2))
    if call != "pair_static":
        case.update(fm_limit=rng.choice((0, 0, 100)), mb_reps=rng.choice((0, 0, 16)),
                    terminals=rng.randrange(2), cut_side=rng.choice((0, 0, 2)))
    else:
        case.update(terminals=rng.randrange(2), alpha=rng.choice((4, 8, 16)))
    if call == "batch" and n <= 1 << 17 and rng.random() < 0.3:
        case.update(mt_alpha=10)
    return case


# ----------------------------------------------------------------- inputs ---

def _csr(n, u, v, seed, whi, device):
    """Symmetric CSR of the undirected edges (u, v), neighbours in ascending order, with edge
    weights in [1, whi]."""
    w = torch.ones_like(u, dtype=torch.int32)
    if whi > 1:
        h = (torch.minimum(u, v) * 0x9E3779B1 + torch.maximum(u, v) * 0x85EBCA77 + seed * 7919)
        h = (h ^ (h >> 15)) * 0x2C1B3C6D
        w = (1 + ((h ^ (h >> 13)) & 0x7FFFFFFF) % whi).to(torch.int32)
    key = torch.cat([u * n + v, v * n + u])
    key, at = torch.sort(key)
    src = torch.div(key, n, rounding_mode="floor")
    xadj = torch.zeros(n + 1, dtype=torch.int64, device=device)
    xadj[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    w = torch.cat([w, w])[at]
    return (xadj.to(torch.int32), (key - src * n).to(torch.int32), w,
            torch.ones(n, dtype=torch.int32, device=device), src)


def _rgg(n, dim, deg, seed, device):
    """Uniform points in the unit square or cube, ids in cell order, and the edges between
    points closer than the radius of the given mean degree."""
    gen = torch.Generator(device=device).manual_seed(seed)
    side = 1 << SIDE_BITS
    p = torch.randint(side, (n, dim), generator=gen, device=device, dtype=torch.int64)
    vol = {2: math.pi, 3: 4.0 / 3.0 * math.pi}[dim]
    radius = min(0.5, (deg / (vol * n)) ** (1.0 / dim))
    cells = max(1, int(1.0 / radius))
    c = p * cells // side
    cell = c[:, 0]
    for d in range(1, dim):
        cell = cell * cells + c[:, d]
    cell, at = torch.sort(cell, stable=True)
    p, c = p[at], c[at]
    total = cells ** dim
    first = torch.zeros(total + 1, dtype=torch.int64, device=device)
    first[1:] = torch.cumsum(torch.bincount(cell, minlength=total), 0)
    most = int((first[1:] - first[:-1]).max())
    r2 = int(radius * radius * float(side) ** 2)
    ids = torch.arange(n, device=device)
    us, vs = [], []
    # a point's own cell and the half of the neighbouring cells that come later
    steps = [()]
    for _ in range(dim):
        steps = [s + (x,) for s in steps for x in (-1, 0, 1)]
    for s in (s for s in steps if s >= (0,) * dim):
        q = c + torch.tensor(s, device=device)
        ok = ((q >= 0) & (q < cells)).all(1)
        other = q[:, 0]
        for d in range(1, dim):
            other = other * cells + q[:, d]
        other = torch.where(ok, other, torch.zeros_like(other))
        lo = first[other]
        hi = torch.where(ok, first[other + 1], lo)
        if s == (0,) * dim:
            lo = torch.maximum(lo, ids + 1)
        for j in range(most):
            u = ids[lo + j < hi]
            if u.numel() == 0:
                break
            v = lo[u] + j
            near = ((p[u] - p[v]) ** 2).sum(1) <= r2
            us.append(u[near])
            vs.append(v[near])
    return p, torch.cat(us), torch.cat(vs)


def _bisect(p, k):
    """Recursive coordinate bisection into k blocks along the widest axis of each."""
    n = p.shape[0]
    part = torch.zeros(n, dtype=torch.int64, device=p.device)  # first block of a vertex's group
    want = torch.full((n,), k, dtype=torch.int64, device=p.device)  # blocks of its group
    far = 1 << (SIDE_BITS + 1)
    while int(want.max()) > 1:
        ext = []
        for d in range(p.shape[1]):
            hi = torch.full((k,), -1, dtype=torch.int64, device=p.device)
            lo = torch.full((k,), far, dtype=torch.int64, device=p.device)
            hi.scatter_reduce_(0, part, p[:, d], "amax")
            lo.scatter_reduce_(0, part, p[:, d], "amin")
            ext.append(hi - lo)
        axis = torch.stack(ext).argmax(0)[part]
        x = p.gather(1, axis[:, None])[:, 0]
        at = torch.argsort(part * far + x, stable=True)
        size = torch.bincount(part, minlength=k)
        start = torch.cumsum(size, 0) - size
        rank = torch.empty_like(at)
        rank[at] = torch.arange(n, device=p.device)
        rank -= start[part]
        left = want // 2
        right = (want > 1) & (rank >= size[part] * left // want.clamp(min=1))
        part = torch.where(right, part + left, part)
        want = torch.where(want > 1, torch.where(right, want - left, left), want)
    return part


def _noise(n, part, src, dst, frac, gen):
    """Moves a share of the boundary vertices to a neighbouring block."""
    other = torch.where(part[dst] != part[src], part[dst], torch.full_like(src, -1))
    best = torch.full((n,), -1, dtype=torch.int64, device=src.device)
    best.scatter_reduce_(0, src, other, "amax")
    move = (best >= 0) & (torch.rand(n, generator=gen, device=src.device) < frac)
    return torch.where(move, best, part)


def _inputs(case, seed, device):
    n, k = case["n"], case["k"]
    gen = torch.Generator(device=device).manual_seed(seed + 1)
    if case["graph"] == "grid":
        side = math.isqrt(n)
        ids = torch.arange(n, device=device)
        x, y = ids % side, ids // side
        u = torch.cat([ids[x < side - 1], ids[y < side - 1]])
        v = torch.cat([ids[x < side - 1] + 1, ids[y < side - 1] + side])
        part = (x * k // side).to(torch.int64)
    else:
        p, u, v = _rgg(n, case["dim"], case["deg"], seed, device)
        part = _bisect(p, k)
    xadj, adjncy, adjwgt, vwgt, src = _csr(n, u, v, seed, case.get("whi", 1), device)
    part = _noise(n, part, src, adjncy.to(torch.int64), case["noise"], gen)
    return fr.DeviceGraph(n, xadj, adjncy, adjwgt, vwgt), part.to(torch.int32)


def _mlp_inputs(case, seed):
    """Weights, standardised features, labels and costs of n labelled pairs."""
    rng = np.random.default_rng(seed)
    w = []
    for i, o in ((8, 64), (64, 64), (64, 5)):
        w += [rng.normal(0, math.sqrt(2.0 / i), i * o), rng.normal(0, 0.1, o)]
    x = rng.normal(0, 1, (case["n"], 8))
    labels = rng.integers(0, 5, case["n"])
    edges = np.cumsum(rng.uniform(0.05, 0.6, (case["n"], 5)), axis=1)
    loss = rng.poisson(1.0, (case["n"], 5)) * (rng.random((case["n"], 5)) < 0.3)
    return (np.concatenate(w).astype(np.float32), x.astype(np.float32),
            labels.astype(np.int32), (edges + 0.4 * loss).astype(np.float32))


OPTIONS = ("area_mode", "depth", "alpha", "alpha_max", "adaptive", "max_iters", "use_mlp",
           "mb_reps", "fm_limit", "active_blocks", "cut_side", "terminals", "mt_alpha")


class _HostGraph:
    """CSR arrays in host memory, as fr.host_graph_struct takes them."""

    def __init__(self, g):
        for name in ("xadj", "adjncy", "adjwgt", "vwgt"):
            setattr(self, name, getattr(g, name).cpu().numpy())


def prepare(case, seed):
    ctx = fr.Context()
    if case["call"] == "mlp":
        w, x, labels, costs = _mlp_inputs(case, seed)
        fr.fr_mlp_set_weights(ctx, w)
        return dict(case=case, ctx=ctx, x=x, labels=labels, costs=costs)
    graph, start = _inputs(case, seed, "cuda")
    prm = fr.params(mb_seed=1, fm_seed=1, mt_seed=1,
                    **{o: case[o] for o in OPTIONS if o in case})
    if case.get("use_mlp"):
        fr.load_trained_mlp(ctx)
    state = dict(case=case, ctx=ctx, prm=prm)
    if case["call"] == "batch":  # the largest matching of the quotient graph
        edges, colour = fr.fr_quotient_matchings(ctx, graph, start, case["k"])
        state["pairs"] = np.ascontiguousarray(edges[colour == np.bincount(colour).argmax()])
    if case["call"] == "pair_host":
        graph, start = _HostGraph(graph), start.cpu().numpy()
        part = start.copy()
    else:
        part = start.clone()
    state.update(graph=graph, start=start, part=part)
    return state


# ------------------------------------------------------------------- calls ---

def _table(records, fields, rows):
    """Records as an integer table of a fixed number of rows (zeros below the last one): how many
    pairs and solves there are depends on the inputs."""
    t = np.zeros((rows, len(fields)), dtype=np.int64)
    for i, r in enumerate(records):
        t[i] = [r[f] for f in fields]
    return t


def run(state):
    case, ctx = state["case"], state["ctx"]
    if case["call"] == "mlp":
        if case["costs"]:
            loss, grad = fr.fr_mlp_loss_grad_cost(ctx, state["x"], state["costs"])
        else:
            loss, grad = fr.fr_mlp_loss_grad(ctx, state["x"], state["labels"])
        return dict(loss=np.float32(loss), grad=grad)
    graph, part, prm, k = state["graph"], state["part"], state["prm"], case["k"]
    if case["call"] == "pair_host":
        part[:] = state["start"]
    else:
        part.copy_(state["start"])
    if case["call"] in ("pair", "pair_host"):
        res, trace, _ = fr.flow_refine_pair(ctx, graph, part, k, 0, 1, prm)
        return dict(part=part, result=_table([res], RESULT, 1),
                    trace=_table(trace, SOLVE, prm.max_iters))
    if case["call"] == "pair_static":
        res, trace = fr.flow_refine_pair_static(ctx, graph, part, k, 0, 1, prm)
        return dict(part=part, result=_table([res], RESULT, 1),
                    trace=_table(trace, SOLVE, prm.max_iters))
    if case["call"] == "batch":
        res, traces = fr.flow_refine_batch(ctx, graph, part, k, state["pairs"], prm)
        return dict(part=part, result=_table(res, RESULT, k // 2),
                    trace=_table([s for t in traces for s in t], SOLVE, k // 2 * prm.max_iters))
    cut, stats = fr.flow_refine_sweep(ctx, graph, part, k, prm, case["max_sweeps"])
    return dict(part=part, cut=cut, stats=stats)


def work(case):
    if case["call"] == "mlp":
        params = 8 * 64 + 64 + 64 * 64 + 64 + 64 * 5 + 5
        return dict(bytes=4 * (case["n"] * (8 + (5 if case["costs"] else 1)) + 2 * params),
                    flops=6 * case["n"] * params)
    # the graph and the partition read once, the partition written once (whole numbers: no
    # floating-point operations)
    n = case["n"]
    arcs = n * (4.0 if case["graph"] == "grid" else case["deg"])
    return dict(bytes=4 * (n + 1) + 8 * arcs + 4 * n + 8 * n, flops=0)


def exact(case, seed):
    if case["call"] != "mlp":
        return None  # whole numbers
    w, x, labels, costs = _mlp_inputs(case, seed)
    w, x, costs = w.astype(np.float64), x.astype(np.float64), costs.astype(np.float64)
    n = case["n"]
    at = np.cumsum([0, 8 * 64, 64, 64 * 64, 64, 64 * 5, 5])
    w1, b1, w2, b2, w3, b3 = (w[i:j] for i, j in zip(at[:-1], at[1:]))
    w1, w2, w3 = w1.reshape(8, 64), w2.reshape(64, 64), w3.reshape(64, 5)
    h1 = np.maximum(x @ w1 + b1, 0)
    h2 = np.maximum(h1 @ w2 + b2, 0)
    z = h2 @ w3 + b3
    z -= z.max(1, keepdims=True)
    p = np.exp(z)
    p /= p.sum(1, keepdims=True)
    if case["costs"]:
        mean = (p * costs).sum(1, keepdims=True)
        loss, dz = mean.mean(), p * (costs - mean) / n
    else:
        hot = np.zeros_like(p)
        hot[np.arange(n), labels] = 1
        loss, dz = -np.log(p[np.arange(n), labels]).mean(), (p - hot) / n
    d2 = dz @ w3.T * (h2 > 0)
    d1 = d2 @ w2.T * (h1 > 0)
    grad = [x.T @ d1, d1.sum(0), h1.T @ d2, d2.sum(0), h2.T @ dz, dz.sum(0)]
    return dict(loss=np.float64(loss), grad=np.concatenate([g.reshape(-1) for g in grad]))
