"""gve_mlp_loss_grad without a gradient: the loss of the full call bit for bit, from
the forward pass alone (its workspace: weight tiles and one sum per 16 rows, not
the activations and gradients of a training step)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 17, 1025, 65536])
def test_loss_without_gradient(n):
    import torch

    import paper_2608_14112_amd as g
    print(f"mlp loss only rows={n}", flush=True)
    rng = np.random.default_rng(n)
    X = torch.from_numpy(rng.normal(size=(n, 16)).astype(np.float32)).cuda()
    T = torch.from_numpy(rng.normal(size=(n, 11)).astype(np.float32)).cuda()
    ctx = g.Context()
    m = g.MLP(ctx, seed=3)
    before = ctx.stats()["workspace_bytes"]
    L = ctypes.c_double()
    g._check(g._lib.gve_mlp_loss_grad(ctx.handle, m.handle, g._ptr(X), g._ptr(T), n, None,
                                      ctypes.byref(L)), ctx.handle)
    assert ctx.stats()["workspace_bytes"] - before < 400_000
    full, _ = g.mlp_loss_grad(ctx, m, X, T)
    assert L.value == full and np.isfinite(full)
