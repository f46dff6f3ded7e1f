"""The vector-Jacobian product of a single image of 32,768 x 32,768 voxels: 2^24
bricks, where four waves a brick would be more threads than a launch may have
(2^32)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_vjp_of_two_to_the_24_bricks():
    import torch

    import paper_2608_14112_amd as g
    edge = 32768
    print("vjp of 2^24 bricks", flush=True)
    t = np.zeros((11, 4), np.float32)
    t[0] = [10, 20000, 32760, 5]
    t[1] = [10, 31000, 32765, 32000]
    t[3] = 1
    t[7:10] = np.log(1.5)
    t[10] = [1.0, -0.5, 2.0, 0.7]
    up = torch.full((1, edge, edge), 1.0, device="cuda")
    grid = g.Grid(edge, edge, 1)
    ctx = g.Context(k=3.0, brick=8, brick_z=32, deterministic=True)
    v = g.vjp(ctx, g.Params(ctx, 4).upload(t), up, grid).cpu().numpy()
    assert ctx.stats()["n_bricks"] == 1 << 24
    # each primitive by itself, in the part of the image that holds its support
    # (moved to a smaller one; sums of the same terms: 1e-6 of the largest)
    for i in range(4):
        lo = [min(max(int(t[a, i]) // 8 * 8 - 16, 0), edge - 64) for a in range(2)]
        one = t[:, i:i + 1].copy()
        small = g.Grid(64, 64, 1, lo[0], lo[1], 0)
        r = g.vjp(ctx, g.Params(ctx, 1).upload(one), up[:, :64, :64].contiguous(), small)
        r = r.cpu().numpy()[:, 0]
        assert np.abs(v[:, i] - r).max() <= 1e-6 * np.abs(r).max()
