"""What fits the fixed scratch of the allocation-free entry point: the last pair
that has always fitted still does, the next one is refused.  700,640 small
primitives in bricks of 8 x 8 x 8, the first of them moved onto the face between
two bricks, so that each adds one (primitive, brick) pair; with reproducible sums
a pair takes 64 bytes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_capacity_of_the_static_scratch():
    import torch

    import paper_2608_14112_amd as g
    n, fits, nb = 700640, 291564, 16
    b = np.arange(n) % nb ** 3
    t = np.zeros((11, n), np.float32)
    for a, c in enumerate((b % nb, (b // nb) % nb, b // nb ** 2)):
        t[a] = 8 * c + 3.5
    t[3] = 1
    t[7:10] = np.log(0.3)
    t[10] = 1e-3
    movable = np.flatnonzero(b % nb < nb - 1)
    field = torch.zeros(8 * nb, 8 * nb, 8 * nb, device="cuda")
    grad = torch.empty(11, n, device="cuda")
    ctx = g.Context(k=3.0, brick=8, brick_z=8, deterministic=True)
    P = g.Params(ctx, n)
    grid = g.Grid(8 * nb, 8 * nb, 8 * nb)
    t[0, movable[:fits]] += 4.0
    print(f"static capacity {n + fits} pairs", flush=True)
    L = g.loss_grad_static(ctx, P.upload(t), field, grid, grad)
    ref = torch.empty_like(grad)
    assert L == g.loss_grad(ctx, P, field, grid, ref) and torch.equal(grad, ref)
    assert ctx.stats()["n_overlaps"] == n + fits
    t[0, movable[fits]] += 4.0
    with pytest.raises(g.GveError) as e:
        g.loss_grad_static(ctx, P.upload(t), field, grid, grad)
    assert e.value.status == g.UNSUPPORTED
