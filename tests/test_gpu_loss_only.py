"""A loss asked for without its gradient runs the forward pass alone: the same
number, bit for bit, as with the gradient, for every brick shape, split and
schedule, for batches, and with the gradient accumulators left usable."""
import numpy as np
import pytest

from synth import fields as S

pytestmark = pytest.mark.gpu

SHAPES = [(8, 8, 1), (8, 8, 4), (8, 16, 1), (8, 16, 2), (8, 32, 1), (8, 32, 4), (16, 16, 1)]


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


@pytest.mark.parametrize("shape", SHAPES)
def test_loss_without_gradient_is_the_same_loss(shape):
    g, torch = _lib()
    dims, n = (45, 30, 41), 400
    p = S.random_params(n, dims, seed=2, scale_range=(0.6, 4.0)).astype(np.float32)
    grid = g.Grid(*dims)
    field = torch.from_numpy(np.random.default_rng(1).uniform(size=grid.shape)
                             .astype(np.float32)).cuda()
    for sched in (g.SCHED_INDEX, g.SCHED_XCD, g.SCHED_QUEUE):
        print(f"loss only {shape} schedule {sched}", flush=True)
        ctx = g.Context(brick=shape[0], brick_z=shape[1], brick_waves=shape[2], schedule=sched,
                        deterministic=True)
        P = g.Params(ctx, n).upload(p)
        a, b = (torch.empty((11, n), device="cuda") for _ in range(2))
        L = g.loss_grad(ctx, P, field, grid, a)
        assert g.loss_grad(ctx, P, field, grid, None) == L
        assert g.loss_grad(ctx, P, field, grid, b) == L and torch.equal(a, b)


def test_batch_loss_without_gradient():
    g, torch = _lib()
    grids = [g.Grid(20, 33, 40), g.Grid(9, 50, 17)]
    ctx = g.Context()
    b = g.Batch(ctx, grids, [100, 60])
    for i, gr in enumerate(grids):
        n = (100, 60)[i]
        q = S.random_params(n, (gr.nx, gr.ny, gr.nz), seed=i, scale_range=(0.8, 4.0))
        b.set_item(i, g.Params(ctx, n).upload(q.astype(np.float32)))
    fields = torch.rand(int(b.voxel_offsets[-1]), device="cuda")
    print("loss only batch", flush=True)
    grad = torch.empty((11, 160), device="cuda")
    L = g.batch_loss_grad(ctx, b, fields, grad)
    assert np.array_equal(g.batch_loss_grad(ctx, b, fields, None), L)
