"""The queue schedule takes bricks in a loop; bricks without pairs, and bricks with
fewer pairs than waves, must pass through it as any other (values and gradients
bit for bit those of one workgroup per brick)."""
import numpy as np
import pytest

from synth import fields as S

pytestmark = pytest.mark.gpu


# far more bricks than a device holds workgroups (16,384 of 8 x 8 x 8), nearly all
# of them empty, so that every workgroup takes empty bricks one after another;
# then no pair at all
@pytest.mark.parametrize("waves", [1, 2, 4])
@pytest.mark.parametrize("bz", [8, 16, 32])
@pytest.mark.parametrize("n", [40, 1])
def test_empty_bricks_under_the_queue(waves, bz, n):
    import torch

    import paper_2608_14112_amd as g
    print(f"queue empty bricks waves={waves} bz={bz} n={n}", flush=True)
    dims = (256, 256, 32 * bz)
    p = S.random_params(n, (16, 16, 16), seed=n, scale_range=(0.7, 3.0)).astype(np.float32)
    if n == 1:
        p[0] = 1e4  # reaches no brick
    field = torch.from_numpy(np.random.default_rng(bz).uniform(size=dims[::-1])
                             .astype(np.float32)).cuda()
    grid, out = g.Grid(*dims), []
    for sched in (g.SCHED_QUEUE, g.SCHED_INDEX):
        ctx = g.Context(k=3.0, brick=8, brick_z=bz, brick_waves=waves, schedule=sched,
                        deterministic=True)
        P = g.Params(ctx, n).upload(p)
        grad = torch.empty((11, n), device="cuda")
        L = g.loss_grad(ctx, P, field, grid, grad)
        L0 = g.loss_grad(ctx, P, field, grid, None)
        v = g.vjp(ctx, P, field, grid)
        assert ctx.stats()["n_bricks"] == 32 * 32 * 32
        out.append((L, L0, grad.cpu().numpy(), v.cpu().numpy()))
    assert out[0][:2] == out[1][:2]
    assert np.array_equal(out[0][2], out[1][2]) and np.array_equal(out[0][3], out[1][3])
