"""The number of waves that share a brick is chosen by the launch's brick count.
At both sides of every limit the values, gradients and vector-Jacobian products
must be those of the one-wave brick bit for bit (the queue schedule, and for
evaluation a batch past the last limit, never split a brick).  Four waves that
the caller asked for become eight or sixteen in small launches: there only the
order of the forward partial sums differs.
"""
import numpy as np
import pytest

from synth import fields as S

pytestmark = pytest.mark.gpu


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _setup(g, torch, bz, nb, seed):
    """A row of nb bricks, 5 x 8 columns each, one of them with over 512 pairs."""
    dims = (5, 8 * nb - 3, bz)
    n = 1200
    p = S.random_params(n, dims, seed=seed, scale_range=(0.7, 5.0)).astype(np.float32)
    p[1, :700] = np.random.default_rng(seed).uniform(0, 8, 700)
    field = torch.from_numpy(np.random.default_rng(seed + 1).uniform(size=dims[::-1])
                             .astype(np.float32)).cuda()
    return dims, n, p, field


EDGES = [(8, 1), (8, 1024), (8, 1025), (8, 2048), (8, 2049),
         (16, 512), (16, 513), (16, 768), (16, 769), (16, 2048), (16, 2049), (16, 3072), (16, 3073),
         (32, 1), (32, 256), (32, 257), (32, 1024), (32, 1025)]


@pytest.mark.parametrize("bz,nb", EDGES)
def test_split_bricks_equal_one_wave_bricks(bz, nb):
    g, torch = _lib()
    print(f"slice rules bz={bz} bricks={nb}", flush=True)
    dims, n, p, field = _setup(g, torch, bz, nb, nb)
    grid = g.Grid(*dims)
    out = []
    for sched in (g.SCHED_QUEUE, g.SCHED_XCD):
        ctx = g.Context(k=3.0, brick=8, brick_z=bz, deterministic=True, schedule=sched)
        P = g.Params(ctx, n).upload(p)
        grad = torch.empty((11, n), device="cuda")
        L = g.loss_grad(ctx, P, field, grid, grad)
        L0 = g.loss_grad(ctx, P, field, grid, None)
        v = g.vjp(ctx, P, field, grid)
        out.append((L, L0, grad.cpu().numpy(), v.cpu().numpy()))
    assert ctx.stats()["n_bricks"] == nb
    assert out[0][:2] == out[1][:2]
    assert np.array_equal(out[0][2], out[1][2]) and np.array_equal(out[0][3], out[1][3])


@pytest.mark.parametrize("bz,nb", [(8, 1), (8, 1024), (8, 1025), (8, 2048), (8, 2049),
                                   (16, 512), (16, 513), (16, 2048), (16, 2049),
                                   (32, 1), (32, 1024), (32, 1025)])
def test_short_slices_equal_whole_columns(bz, nb):
    g, torch = _lib()
    print(f"slice rules evaluate bz={bz} bricks={nb}", flush=True)
    dims, n, p, _ = _setup(g, torch, bz, nb, nb)
    ctx = g.Context(k=3.0, brick=8, brick_z=bz)
    P = g.Params(ctx, n).upload(p)
    alone = g.evaluate(ctx, P, g.Grid(*dims)).cpu().numpy().ravel()
    big = g.Grid(264, 264, 320)
    Q = g.Params(ctx, 50).upload(S.random_params(50, (264, 264, 320), seed=4,
                                                 scale_range=(2.0, 6.0)).astype(np.float32))
    b = g.Batch(ctx, [g.Grid(*dims), big], [n, 50])
    b.set_item(0, P)
    b.set_item(1, Q)
    both = g.batch_evaluate(ctx, b).cpu().numpy()
    assert np.array_equal(both[:alone.size], alone)


@pytest.mark.parametrize("bz,nb", [(8, 1), (8, 128), (8, 129), (8, 2048), (16, 512), (16, 513),
                                   (16, 2049), (32, 3), (32, 768), (32, 769)])
def test_more_waves_than_asked_for(bz, nb):
    """Against one wave: a voxel's sum of up to 1,200 terms is formed from 4 .. 16
    partial sums, so it moves by at most 1,200 roundings of its terms' magnitudes,
    in practice a few; the gradient follows the residual linearly.  1e-5 of the
    largest gradient of each row covers 80 roundings."""
    g, torch = _lib()
    print(f"waves 4 bz={bz} bricks={nb}", flush=True)
    dims, n, p, field = _setup(g, torch, bz, nb, nb)
    out = []
    for waves in (1, 4):
        ctx = g.Context(k=3.0, brick=8, brick_z=bz, deterministic=True, brick_waves=waves)
        P = g.Params(ctx, n).upload(p)
        grad = torch.empty((11, n), device="cuda")
        L = g.loss_grad(ctx, P, field, g.Grid(*dims), grad)
        L0 = g.loss_grad(ctx, P, field, g.Grid(*dims), None)
        assert L == L0
        out.append((L, grad.cpu().numpy().astype(np.float64)))
    assert abs(out[0][0] - out[1][0]) <= 1e-5 * out[0][0]
    d, ref = np.abs(out[0][1] - out[1][1]).max(1), np.abs(out[0][1]).max(1)
    assert np.all(d <= 1e-5 * ref), (d / ref)
