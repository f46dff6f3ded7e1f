"""brick_waves fixes the partial sums that a voxel's value is formed from.  A launch
of few bricks runs more waves than that, the queue schedule and larger launches do
not: the three schedules, and a volume alone or beside a large one, must give the
same bits (reproducible sums, equality, no tolerance)."""
import numpy as np
import pytest

from synth import fields as S

pytestmark = pytest.mark.gpu


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _inputs(torch, dims, n, seed, crowd=0):
    p = S.random_params(n, dims, seed=seed, scale_range=(0.7, 5.0)).astype(np.float32)
    if crowd:  # more pairs in one brick than a brick records (512)
        p[1, :crowd] = np.random.default_rng(seed).uniform(0, 8, crowd)
    field = np.random.default_rng(seed + 1).uniform(size=dims[::-1]).astype(np.float32)
    return p, torch.from_numpy(field).cuda()


def _results(g, torch, ctx, p, field, grid):
    P = g.Params(ctx, p.shape[1]).upload(p)
    grad = torch.empty((11, p.shape[1]), device="cuda")
    L = g.loss_grad(ctx, P, field, grid, grad)
    return L, g.loss_grad(ctx, P, field, grid, None), grad.cpu().numpy()


# both sides of every limit; fewer pairs than shares; bricks past 512 pairs
@pytest.mark.parametrize("bz,nb,n", [
    (8, 1, 3), (8, 128, 1200), (8, 129, 1200), (8, 2048, 1200), (8, 8192, 1200), (8, 8193, 1200),
    (16, 1, 3), (16, 512, 1200), (16, 513, 1200), (16, 4096, 1200), (16, 4097, 1200),
    (32, 1, 3), (32, 3, 1200), (32, 512, 1200), (32, 513, 1200), (32, 4096, 1200),
    (32, 4097, 1200)])
@pytest.mark.parametrize("waves", [2, 4])
def test_schedules_agree(bz, nb, n, waves):
    g, torch = _lib()
    print(f"wave order bz={bz} bricks={nb} n={n} waves={waves}", flush=True)
    dims = (5, 8 * nb - 3, bz)
    p, field = _inputs(torch, dims, n, nb, crowd=700 if n > 700 else 0)
    out = []
    for sched in (g.SCHED_QUEUE, g.SCHED_INDEX, g.SCHED_XCD):
        ctx = g.Context(k=3.0, brick=8, brick_z=bz, deterministic=True, brick_waves=waves,
                        schedule=sched)
        out.append(_results(g, torch, ctx, p, field, g.Grid(*dims)))
        assert ctx.stats()["n_bricks"] == nb and ctx.stats()["bin_waves"] == waves
    assert out[0][0] == out[0][1]
    for o in out[1:]:
        assert o[:2] == out[0][:2] and np.array_equal(o[2], out[0][2])


@pytest.mark.parametrize("bz", [8, 16, 32])
@pytest.mark.parametrize("waves", [2, 4])
def test_batch_equals_volume_alone(bz, waves):
    g, torch = _lib()
    print(f"wave order batch bz={bz} waves={waves}", flush=True)
    dims, big, n = (37, 29, 70), (264, 264, 264), 900
    p, field = _inputs(torch, dims, n, 5)
    q, other = _inputs(torch, big, 400, 6)
    ctx = g.Context(k=3.0, brick=8, brick_z=bz, deterministic=True, brick_waves=waves)
    L, L0, grad = _results(g, torch, ctx, p, field, g.Grid(*dims))
    b = g.Batch(ctx, [g.Grid(*dims), g.Grid(*big)], [n, 400])
    b.set_item(0, g.Params(ctx, n).upload(p))
    b.set_item(1, g.Params(ctx, 400).upload(q))
    both = torch.empty((11, n + 400), device="cuda")
    losses = g.batch_loss_grad(ctx, b, torch.cat([field.ravel(), other.ravel()]), both)
    assert ctx.stats()["n_bricks"] > (8192 if bz < 32 else 4096)
    assert losses[0] == L == L0
    assert np.array_equal(both.cpu().numpy()[:, :n], grad)
