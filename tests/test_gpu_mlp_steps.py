"""An epoch of training is its batches: rows in the seeded order, standardised with
the whole set's statistics, one Adam step each, a short last batch as any other.
The expected losses and weights are formed batch by batch from gve_mlp_loss_grad,
the oracle's permutation and Adam on the host."""
import numpy as np
import pytest

from oracle import mlp as Mo

pytestmark = pytest.mark.gpu

# two splits of the weight gradients, then 512 rows in one; short batches and a
# last one of a single row; one batch
CASES = [(1537, 1025), (200, 33), (33, 16), (70, 70)]


def _setup(n, seed):
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    rng = np.random.default_rng(seed)
    X = rng.normal(0.5, 2.0, size=(n, 16)).astype(np.float32)
    T = (rng.normal(size=(n, 11)) * 0.3 - 0.2).astype(np.float32)
    return g, torch, X, T


def _standardised(flat, X, T, g):
    st = flat[g.MLP_NWEIGHT:]
    return (X - st[:16]) / st[16:32], (T - st[32:43]) / st[43:54]


def _batches(n, batch, seed, epoch):
    perm = Mo.epoch_permutation(n, seed, epoch)
    return [perm[a:a + batch] for a in range(0, n, batch)]


@pytest.mark.parametrize("n,batch", CASES)
def test_epoch_loss_is_the_mean_of_its_batches(n, batch):
    """Learning rate 0.  The same kernel on the same rows: equal up to the order of
    the float64 sums (1e-12)."""
    g, torch, X, T = _setup(n, n)
    print(f"mlp epoch loss rows={n} batch={batch}", flush=True)
    ctx = g.Context()
    m = g.MLP(ctx, seed=2)
    h = g.mlp_train(ctx, m, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), epochs=2,
                    batch=batch, lr=0.0, seed=9)
    Xs, Ts = _standardised(m.export(), X, T, g)
    for ep in range(2):
        losses = [g.mlp_loss_grad(ctx, m, torch.from_numpy(Xs[r]).cuda(),
                                  torch.from_numpy(Ts[r]).cuda())[0]
                  for r in _batches(n, batch, 9, ep)]
        assert abs(h[ep] - np.mean(losses)) <= 1e-12 * h[ep]


@pytest.mark.parametrize("n,batch", CASES)
def test_epochs_are_single_steps(n, batch):
    """Two epochs against a gradient and a host Adam step per batch.  Weights that
    differ in the last place of float32 rarely round to another bfloat16 (one in
    2^16, by 2^-8), so the paths stay together: 1e-3 of the distance covered."""
    g, torch, X, T = _setup(n, n + 1)
    print(f"mlp steps rows={n} batch={batch}", flush=True)
    ctx = g.Context()
    m, ref = g.MLP(ctx, seed=4), g.MLP(ctx, seed=4)
    flat = ref.export()
    start = flat[:g.MLP_NWEIGHT].copy()
    lr = 1e-3
    h = g.mlp_train(ctx, m, torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), epochs=2,
                    batch=batch, lr=lr, seed=7)
    Xs, Ts = _standardised(m.export(), X, T, g)
    mm = np.zeros(g.MLP_NWEIGHT)
    vv = np.zeros(g.MLP_NWEIGHT)
    t = 0
    for ep in range(2):
        losses = []
        for r in _batches(n, batch, 7, ep):
            ref.load(flat)
            L, gr = g.mlp_loss_grad(ctx, ref, torch.from_numpy(Xs[r]).cuda(),
                                    torch.from_numpy(Ts[r]).cuda())
            gr = gr.cpu().numpy().astype(np.float64)
            t += 1
            mm = 0.9 * mm + 0.1 * gr
            vv = 0.999 * vv + 0.001 * gr * gr
            flat[:g.MLP_NWEIGHT] -= lr * (mm / (1 - 0.9 ** t)) / (
                np.sqrt(vv / (1 - 0.999 ** t)) + 1e-8)
            losses.append(L)
        assert abs(h[ep] - np.mean(losses)) <= 1e-4 * h[ep]
    moved = flat[:g.MLP_NWEIGHT] - start
    assert np.linalg.norm(moved) > 0
    got = m.export()[:g.MLP_NWEIGHT] - start
    assert np.linalg.norm(got - moved) <= 1e-3 * np.linalg.norm(moved)
