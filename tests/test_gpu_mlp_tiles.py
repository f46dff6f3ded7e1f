"""The network's kernels at the edges of their tiles: rows that do not fill a
16-row training tile or a 64-row inference step, batches on both sides of the
split of the weight gradients (1,024 rows), and training against single steps.

Tolerances are those of the bfloat16 oracle's comparison: an activation that
lands near a rounding boundary may round the other way on one side (2^-9 of one
term), so outputs agree to 1e-3 and gradients to 1e-2 norm-wise per tensor.
"""
import numpy as np
import pytest

from oracle import mlp as Mo

pytestmark = pytest.mark.gpu


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _net(g, ctx, seed):
    p = Mo.init_params(seed)
    rng = np.random.default_rng(seed + 1)
    for k in ("b1", "b2", "b3"):
        p[k] = rng.normal(0, 0.1, size=p[k].shape)
    flat = np.concatenate([p[k].ravel() for k in ("W1", "b1", "W2", "b2", "W3", "b3")] +
                          [np.zeros(16), np.ones(16), np.zeros(11), np.ones(11)])
    m = g.MLP(ctx, seed=0)
    m.load(flat.astype(np.float32))
    return m, {k: v.astype(np.float32).astype(np.float64) for k, v in p.items()}


@pytest.mark.parametrize("n", [1, 15, 16, 17, 1024, 1025, 1537])
def test_gradient_at_tile_and_split_edges(n):
    g, torch = _lib()
    print(f"mlp_loss_grad rows={n}", flush=True)
    ctx = g.Context()
    m, p = _net(g, ctx, 5)
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, 16)).astype(np.float32)
    T = rng.normal(size=(n, 11)).astype(np.float32)
    L, grad = g.mlp_loss_grad(ctx, m, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda())
    grad = grad.cpu().numpy().astype(np.float64)
    Lr, gr = Mo.loss_and_grads(p, X.astype(np.float64), T.astype(np.float64), bf16=True)
    assert abs(L - Lr) <= 1e-3 * Lr
    off = 0
    for name, shape in g.MLP_LAYOUT:
        size = int(np.prod(shape))
        assert np.linalg.norm(grad[off:off + size] - gr[name].ravel()) <= \
            1e-2 * np.linalg.norm(gr[name]), name
        off += size


@pytest.mark.parametrize("n", [63, 64, 65, 65537])
def test_inference_at_step_edges(n):
    g, torch = _lib()
    print(f"mlp_forward rows={n}", flush=True)
    ctx = g.Context()
    m, p = _net(g, ctx, 3)
    X = np.random.default_rng(n).normal(size=(n, 16)).astype(np.float32)
    out = torch.full((n + 1, 11), 7.0, device="cuda")  # a row past the end stays untouched
    Xt = torch.from_numpy(X).cuda()
    Y = g.mlp_forward(ctx, m, Xt)
    g._check(g._lib.gve_mlp_forward(ctx.handle, m.handle, g._ptr(Xt), n, g._ptr(out)), ctx.handle)
    assert torch.equal(out[:n], Y) and bool((out[n] == 7.0).all())
    Yr, _ = Mo.forward(p, X.astype(np.float64), bf16=True)
    assert np.linalg.norm(Y.cpu().numpy() - Yr) <= 1e-3 * np.linalg.norm(Yr)


def test_last_partial_batch():
    """An epoch of 1,537 rows in batches of 1,025 (two splits, then 512 rows in
    one): a zero learning rate leaves the weights, and the mean of the batch
    losses over the permuted rows is the whole set's up to the batch sizes."""
    g, torch = _lib()
    ctx = g.Context()
    m, _ = _net(g, ctx, 4)
    rng = np.random.default_rng(0)
    X = torch.from_numpy(rng.normal(size=(1537, 16)).astype(np.float32)).cuda()
    T = torch.from_numpy(rng.normal(size=(1537, 11)).astype(np.float32)).cuda()
    before = m.export()[:g.MLP_NWEIGHT]
    print("mlp_train rows=1537 batch=1025 lr=0", flush=True)
    h = g.mlp_train(ctx, m, X, T, epochs=2, batch=1025, lr=0.0, seed=1)
    assert np.array_equal(m.export()[:g.MLP_NWEIGHT], before)
    assert np.all(np.isfinite(h)) and abs(h[0] - h[1]) < 0.1 * h[0]
