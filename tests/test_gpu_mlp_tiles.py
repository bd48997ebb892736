"""The network's loss and gradient at the edges of the 64-sample tiles (one
sample, one short of and one past a tile, one past four tiles, many tiles)
against the float64 oracle.

Tolerance: every value is a chain of at most 8 + 64 + 5 + 64 products forward
and back and a sum of at most 64 + tiles / 4 + 4 terms; at 6e-8 per rounding,
300 of them stay below 2e-5 of the largest gradient entry."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context()
    yield c
    c.close()


@pytest.mark.parametrize("with_costs", [False, True])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 5000])
def test_gradient_at_tile_edges(gpu_lib, ctx, n, with_costs):
    fr = gpu_lib
    rng = np.random.default_rng(n)
    fr.fr_mlp_init(ctx, 40 + n)
    P = {k: v.astype(np.float64) for k, v in fr.mlp_unpack(fr.fr_mlp_get_weights(ctx)).items()}
    x = rng.normal(0, 1, (n, 8)).astype(np.float32)
    if with_costs:
        y = rng.uniform(0, 4, (n, 5)).astype(np.float32)
        loss, grad = fr.fr_mlp_loss_grad_cost(ctx, x, y)
        l_ref, g_ref = oracle.mlp_loss_grad_cost(P, x.astype(np.float64), y.astype(np.float64))
    else:
        y = rng.integers(0, 5, n).astype(np.int32)
        loss, grad = fr.fr_mlp_loss_grad(ctx, x, y)
        l_ref, g_ref = oracle.mlp_loss_grad(P, x.astype(np.float64), y)
    ref = np.concatenate([g_ref[k].reshape(-1) for k in ("W1", "b1", "W2", "b2", "W3", "b3")])
    print(f"mlp tiles n={n} costs={with_costs}: loss {loss} ref {l_ref}, grad off "
          f"{np.abs(grad - ref).max() / np.abs(ref).max():.2e}", flush=True)
    assert abs(loss - l_ref) <= 2e-5 * abs(l_ref)
    assert np.abs(grad - ref).max() <= 2e-5 * np.abs(ref).max()
