"""The allocation's common weight factor kappa = <V, U> / <U, U> is summed inside
the field pass, brick by brick.  The allocated field must then be its own best
fit, <V, Vhat> = <Vhat, Vhat>, whatever the brick shape and whether bricks are
sliced.  Weights are rounded to float32 and the field sums of them are float32,
a few roundings of 6e-8 in a ratio of sums of like sign: 1e-6.
"""
import numpy as np
import pytest


pytestmark = pytest.mark.gpu


# one slab of short slices; ragged; slices of 4 and 8; past the sliced launches
@pytest.mark.parametrize("dims,budget", [((24, 17, 9), 40), ((61, 45, 37), 300),
                                         ((130, 97, 101), 900), ((203, 211, 260), 2500)])
def test_allocated_field_is_its_own_best_fit(dims, budget):
    import torch

    import paper_2608_14112_amd as g
    f = torch.from_numpy(_blobs(dims)).cuda()
    kappas = []
    for brick, bz in ((8, 8), (8, 16), (8, 32), (16, 16)):
        print(f"kappa {dims} brick {brick}x{bz}", flush=True)
        ctx = g.Context(k=3.0, brick=brick, brick_z=bz)
        P, info = g.allocate(ctx, f, g.Grid(*dims), budget, 5)
        v = g.evaluate(ctx, P, g.Grid(*dims)).double()
        ratio = float((v * f.double()).sum() / (v * v).sum())
        assert abs(ratio - 1.0) <= 1e-6
        kappas.append(info["kappa"])
    assert np.allclose(kappas, kappas[0], rtol=1e-6)


def _blobs(dims):
    """Smooth blobs in [0, 1], mostly occupied."""
    rng = np.random.default_rng(7)
    z, y, x = (np.arange(n, dtype=np.float64) for n in dims[::-1])
    f = np.zeros(dims[::-1])
    for _ in range(6):
        c = [rng.uniform(0, n) for n in dims]
        s = [0.15 * n + 1.5 for n in dims]
        e = [np.exp(-0.5 * ((q - m) / w) ** 2) for q, m, w in zip((x, y, z), c, s)]
        f += rng.uniform(0.4, 1.0) * e[2][:, None, None] * e[1][:, None] * e[0]
    return (f / f.max()).astype(np.float32)
