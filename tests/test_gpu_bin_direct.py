"""Small sets are binned by one kernel that tests every (brick, primitive) pair;
the queue schedule always takes the general binning (scans, cull, sort).  Both
list the same pairs in the same order, so the field, the support counts and the
pair and degenerate-quaternion counts are equal (no tolerance).
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


# (grid, primitives, scales): runs of 64 and passes of 2,048 primitives, each
# one short, whole and one over; a single voxel column; the largest directly
# binned volume (32,768 primitives) and the first that is not, the most bricks
# (16,384 of 8 x 8 x 8) and one more; ragged extents
CASES = [((1, 1, 9), 1, (0.5, 2.0)),
         ((16, 16, 16), 63, (1.0, 3.0)),
         ((17, 9, 33), 64, (1.0, 6.0)),
         ((30, 24, 20), 65, (4.0, 12.0)),
         ((64, 64, 64), 2047, (1.5, 4.0)),
         ((64, 64, 64), 2048, (1.5, 4.0)),
         ((61, 45, 37), 2049, (0.5, 8.0)),
         ((40, 24, 41), 32768, (0.5, 3.0)),
         ((40, 24, 41), 32769, (0.5, 3.0)),
         ((256, 256, 128), 300, (0.5, 6.0)),
         ((8, 8, 131073), 300, (0.5, 6.0))]


def _params(n, dims, seed, scales):
    p = S.random_params(n, dims, seed=seed, scale_range=scales).astype(np.float32)
    if n >= 63:
        p[3:7, 3] = 0.0           # degenerate quaternion
        p[0, 5] = -1e4            # boxes that miss the volume, on both sides
        p[2, 62] = 1e4
    return p


@pytest.mark.parametrize("brick,brick_z", [(8, 8), (8, 32), (16, 16)])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_direct_binning_equals_general(case, brick, brick_z):
    g, torch = _lib()
    dims, n, scales = CASES[case]
    print(f"direct binning {dims} n={n} brick={brick}x{brick_z}", flush=True)
    p = _params(n, dims, case, scales)
    grid = g.Grid(*dims, 1, -2, 3) if case % 2 else g.Grid(*dims)
    if case % 2:
        p[:3] += np.float32([[1], [-2], [3]])
    out = []
    for sched in (g.SCHED_QUEUE, g.SCHED_INDEX, g.SCHED_XCD):
        ctx = g.Context(k=3.0, brick=brick, brick_z=brick_z, schedule=sched)
        P = g.Params(ctx, n).upload(p)
        got = []
        for _ in range(3):        # the count slots are used in turn
            f = g.evaluate(ctx, P, grid).cpu().numpy()
            st = ctx.stats()
            got.append((f, st["n_overlaps"], st["n_degenerate_q"], st["n_bricks"]))
        assert all(np.array_equal(f[0], got[0][0]) and f[1:] == got[0][1:] for f in got)
        out.append(got[0] + (g.count_pairs(ctx, P, grid),))
    for o in out[1:]:
        assert np.array_equal(o[0], out[0][0])
        assert o[1:] == out[0][1:]
    assert out[0][2] == (1 if n >= 63 else 0)


def test_direct_binning_of_a_batch():
    g, torch = _lib()
    dims = [(9, 8, 8), (40, 33, 20), (1, 1, 1), (16, 64, 24), (24, 24, 24)]
    counts = [1, 700, 1, 65, 2200]
    params = [S.random_params(c, d, seed=i, scale_range=(1.0, 4.0)).astype(np.float32)
              for i, (d, c) in enumerate(zip(dims, counts))]
    out = []
    for sched in (g.SCHED_QUEUE, g.SCHED_XCD):
        ctx = g.Context(k=3.0, brick=8, brick_z=16, schedule=sched)
        b = g.Batch(ctx, [g.Grid(*d) for d in dims], counts)
        for i, p in enumerate(params):
            b.set_item(i, g.Params(ctx, counts[i]).upload(p))
        f = [x.cpu().numpy() for x in g.batch_evaluate(ctx, b)]
        out.append((f, ctx.stats()["n_overlaps"], g.batch_count_pairs(ctx, b)))
    assert all(np.array_equal(a, b) for a, b in zip(out[0][0], out[1][0]))
    assert out[0][1:] == out[1][1:]


@pytest.mark.parametrize("iters", [1, 5])
def test_refinement_binned_directly(iters):
    """The counts after a refinement are those of binning its last start afresh,
    and the two binnings' trajectories differ by the order of float atomics only:
    every Adam step moves a parameter by at most about lr, and only a gradient
    sum whose sign depends on that order can make two steps differ, so the mean
    difference is held to a hundredth of what lr allows."""
    g, torch = _lib()
    dims, n, lr = (40, 33, 47), 500, 1e-3
    p = S.random_params(n, dims, seed=4, scale_range=(1.5, 4.0)).astype(np.float32)
    f = torch.from_numpy(np.random.default_rng(1).uniform(size=dims[::-1]).astype(np.float32)).cuda()
    res = []
    for sched in (g.SCHED_QUEUE, g.SCHED_XCD):
        ctx = g.Context(k=3.0, lr=lr, brick=8, brick_z=16, schedule=sched)
        P = g.Params(ctx, n).upload(p)
        L = g.refine(ctx, P, f, g.Grid(*dims), iters)
        st = ctx.stats()
        assert st["n_resized"] == 0 and st["n_degenerate_q"] == 0
        res.append((L, P.download(), st["n_overlaps"]))
    assert np.allclose(res[0][0], res[1][0], rtol=1e-5 * iters)
    assert np.abs(res[0][1] - res[1][1]).mean() <= 0.01 * lr * iters
    if iters == 1:
        assert res[0][2] == res[1][2] > 0
