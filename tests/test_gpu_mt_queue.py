"""The queue of the multi-try searches where its handling changes: more
entries than a request answers, than one scan takes (1,024), than its local
store (2,048) and than its group bounds (65,536) hold; and gains of vertices
whose arcs no longer fit a lane group's registers (32)."""
import numpy as np
import pytest

from tests.helpers import csr_from_edges
from tests.test_gpu_mt import _batch_vs_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.close()


def _params(seed):
    return dict(area_mode=0, depth=0, alpha=1, alpha_max=1, adaptive=0, max_iters=1,
                eps_ppm=1_000_000, mt_alpha=1_000_000, mt_seed=seed)


@pytest.mark.parametrize("leaves", [15, 63, 64, 1022, 1023, 1024, 2046, 2047, 2048, 65535, 65536, 70000])
def test_queue_of_a_star(gpu_lib, ctx, leaves):
    """A hub whose leaves are in three other blocks: its search queues the
    leaves together and pops them all (no stopping rule applies)."""
    rng = np.random.default_rng(leaves)
    hub = leaves
    edges = [(i, hub) for i in range(leaves)]
    w = rng.integers(1, 4, leaves).tolist()
    g = csr_from_edges(leaves + 1, edges, w)
    part = rng.integers(0, 4, leaves + 1).astype(np.int32)
    part[hub] = 0
    _batch_vs_oracle(gpu_lib, ctx, g, part, 4, [(0, 1)], _params(leaves))


@pytest.mark.parametrize("deg", [15, 16, 17, 31, 32, 33, 63, 64, 65, 200])
def test_degrees(gpu_lib, ctx, deg):
    """A circulant graph of degree 2 * (deg // 2) with chords to make the odd
    degrees, six blocks at random: every gain is one of that many arcs."""
    n = 600
    rng = np.random.default_rng(deg)
    edges = {(i, (i + d) % n) for i in range(n) for d in range(1, deg // 2 + 1)}
    if deg % 2:
        edges |= {(i, i + n // 2) for i in range(n // 2)}
    edges = sorted((min(e), max(e)) for e in edges)
    g = csr_from_edges(n, edges, rng.integers(1, 5, len(edges)).tolist())
    part = rng.integers(0, 6, n).astype(np.int32)
    p = dict(_params(deg), mt_alpha=10)
    _batch_vs_oracle(gpu_lib, ctx, g, part, 6, [(0, 1), (2, 3)], p)


@pytest.mark.parametrize("k", [2048, 2049])
def test_many_blocks(gpu_lib, ctx, k):
    """Block weights in the local store and beyond it."""
    n = 6 * k
    rng = np.random.default_rng(k)
    edges = sorted({(i, i + 1) for i in range(n - 1)} | {(i, i + 97) for i in range(n - 97)})
    g = csr_from_edges(n, edges, rng.integers(1, 5, len(edges)).tolist())
    part = (np.arange(n) // 6).astype(np.int32)
    swap = rng.permutation(n)[: n // 5]
    part[swap] = rng.permutation(part[swap])
    p = dict(_params(k), mt_alpha=10, eps_ppm=300_000)
    _batch_vs_oracle(gpu_lib, ctx, g, part, k, [(0, 1), (2, 3), (4, 5)], p)
