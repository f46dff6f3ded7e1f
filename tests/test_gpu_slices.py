"""Bricks whose offsets are dealt to several waves must give the unsliced results
bit for bit: each voxel's value and each pair's gradient sums are formed from the
same operations in the same order.

The queue schedule never slices, brick order and XCD chunks slice launches of at
most 12,288 bricks (evaluation: 10,240), so the schedules and a batch past the
limit are the two sides of each comparison (reproducible sums, equality, no
tolerance).
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


# (grid, primitives, scales): ragged in every axis; a single column; more than
# 512 pairs in a brick (the recorded offsets end there); wide primitives
CASES = [((37, 29, 70), 300, (0.6, 4.0)),
         ((1, 1, 9), 5, (0.5, 2.0)),
         ((24, 17, 33), 900, (2.0, 5.0)),
         ((40, 40, 64), 60, (8.0, 20.0))]


@pytest.mark.parametrize("brick_z", [16, 32])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_sliced_fused_pass_equals_unsliced(brick_z, case):
    g, torch = _lib()
    dims, n, sr = CASES[case]
    print(f"slices {dims} n={n} bz={brick_z}", flush=True)
    p = S.random_params(n, dims, seed=case, scale_range=sr).astype(np.float32)
    grid = g.Grid(*dims)
    field = torch.from_numpy(np.random.default_rng(case).uniform(size=grid.shape)
                             .astype(np.float32)).cuda()
    out = []
    for sched in (g.SCHED_QUEUE, g.SCHED_INDEX, g.SCHED_XCD):
        ctx = g.Context(k=3.0, brick=8, brick_z=brick_z, deterministic=True, schedule=sched)
        P = g.Params(ctx, n).upload(p)
        grad = torch.empty((11, n), device="cuda")
        L = g.loss_grad(ctx, P, field, grid, grad)
        L0 = g.loss_grad(ctx, P, field, grid, None)
        v = g.vjp(ctx, P, field, grid)
        out.append((L, L0, grad.cpu().numpy(), v.cpu().numpy()))
    for o in out[1:]:
        assert o[0] == out[0][0] and o[1] == out[0][1]
        assert np.array_equal(o[2], out[0][2]) and np.array_equal(o[3], out[0][3])
    assert out[0][0] == out[0][1]


@pytest.mark.parametrize("brick_z", [16, 32])
def test_sliced_evaluation_equals_unsliced(brick_z):
    """A volume alone (sliced) and beside one that takes the launch past the
    limit (unsliced)."""
    g, torch = _lib()
    dims, n, sr = CASES[0]
    p = S.random_params(n, dims, seed=3, scale_range=sr).astype(np.float32)
    p[10, 7] = np.inf  # reaches the voxels of its own box only
    big = g.Grid(264, 264, 320)
    q = S.random_params(50, (264, 264, 320), seed=4, scale_range=(2.0, 6.0)).astype(np.float32)
    ctx = g.Context(k=3.0, brick=8, brick_z=brick_z)
    print(f"slices evaluate bz={brick_z}", flush=True)
    P = g.Params(ctx, n).upload(p)
    alone = g.evaluate(ctx, P, g.Grid(*dims)).cpu().numpy().ravel()
    Q = g.Params(ctx, 50).upload(q)
    b = g.Batch(ctx, [g.Grid(*dims), big], [n, 50])
    b.set_item(0, P)
    b.set_item(1, Q)
    both = g.batch_evaluate(ctx, b).cpu().numpy()
    assert np.array_equal(both[:alone.size], alone, equal_nan=True)
