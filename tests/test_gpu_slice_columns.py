"""A brick at the volume's edge has columns outside it.  A pair that reaches only
such columns is skipped whole, however the brick is split, so that an infinite
weight reaches the same voxels: those of the one-wave brick (queue schedule; for
evaluation a batch past every limit), bit for bit.

The primitives below were found by a search over random frames on the CPU: with
k = 3 in a volume of 10 x 8 x 32 they have no voxel in the second brick's inside
columns (x = 8, 9), by a margin of 2 % in m^2, though their boxes and the
separating-plane test keep the pair, and some in its outside columns; or they
have inside voxels, but none at some offsets where they reach outside columns.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DIMS = (10, 8, 32)
OUTSIDE = [  # mu, q, log-scales
    [12.398, 1.1411, 24.9994, 0.7086, -0.5408, 0.1957, -0.4087, 0.0035, -1.5666, 0.5508],
    [11.9698, 5.6509, 20.7715, 0.1776, 0.6227, 0.0867, -0.757, 0.3177, -1.747, 0.2727],
    [12.0854, 5.4363, 18.8929, 0.8812, 0.1108, 0.4072, -0.213, 0.5211, -0.4959, -1.2237]]
ACROSS = [
    [11.9543, 5.9635, 11.9092, -0.4111, 0.3625, -0.8174, -0.1773, 1.2834, -1.204, -0.9163],
    [9.7904, 5.4622, 13.1665, 0.8905, -0.0268, -0.4529, -0.0338, 1.034, -1.204, -0.9163]]


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _theta(prim, weight):
    """The primitive with the given weight beside one that covers the edge."""
    t = np.zeros((11, 2), np.float32)
    t[:10, 0] = prim
    t[10, 0] = weight
    t[:, 1] = [7, 4, 16, 1, 0, 0, 0, 1.0, 1.0, 1.5, 0.5]
    return t


@pytest.mark.parametrize("bz", [8, 16, 32])
@pytest.mark.parametrize("i", range(len(OUTSIDE) + len(ACROSS)))
def test_evaluation(i, bz):
    g, torch = _lib()
    print(f"slice columns evaluate {i} bz={bz}", flush=True)
    ctx = g.Context(k=3.0, brick=8, brick_z=bz)
    P = g.Params(ctx, 2).upload(_theta((OUTSIDE + ACROSS)[i], np.inf))
    alone = g.evaluate(ctx, P, g.Grid(*DIMS)).cpu().numpy().ravel()
    big = g.Grid(264, 264, 320)
    t = np.zeros((11, 1), np.float32)
    t[:4, 0] = [130, 130, 160, 1]
    b = g.Batch(ctx, [g.Grid(*DIMS), big], [2, 1])
    b.set_item(0, P)
    b.set_item(1, g.Params(ctx, 1).upload(t))
    both = g.batch_evaluate(ctx, b).cpu().numpy()
    assert np.array_equal(both[:alone.size], alone, equal_nan=True)
    assert np.isfinite(alone).all() == (i < len(OUTSIDE))


@pytest.mark.parametrize("waves", [1, 4])
@pytest.mark.parametrize("bz", [8, 16, 32])
@pytest.mark.parametrize("i", range(len(OUTSIDE)))
def test_loss_and_gradient(i, bz, waves):
    g, torch = _lib()
    print(f"slice columns loss {i} bz={bz} waves={waves}", flush=True)
    field = torch.from_numpy(np.random.default_rng(i).uniform(size=DIMS[::-1])
                             .astype(np.float32)).cuda()
    out = []
    for sched in (g.SCHED_QUEUE, g.SCHED_XCD):
        ctx = g.Context(k=3.0, brick=8, brick_z=bz, brick_waves=waves, schedule=sched,
                        deterministic=True)
        P = g.Params(ctx, 2).upload(_theta(OUTSIDE[i], np.inf))
        grad = torch.empty((11, 2), device="cuda")
        L = g.loss_grad(ctx, P, field, g.Grid(*DIMS), grad)
        assert np.isfinite(L) and L == g.loss_grad(ctx, P, field, g.Grid(*DIMS), None)
        out.append((L, grad.cpu().numpy()))
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1], equal_nan=True)
