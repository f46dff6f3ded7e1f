"""Box means and variances come from prefix sums within blocks of 64 x 8 x 8
voxels, or from summed-area tables of the volume where the set's boxes touch too
many blocks (more than two for each voxel).  Adding many wide primitives to a set
moves it from the first way to the second; both against the oracle.

Both ways sum in double; a table entry is at most the whole volume's sum, so a
box sum from eight of them is off by some 8 * 2^-52 of that, under 1e-11 of a
mean here, and what is compared is float32: two roundings.
"""
import numpy as np
import pytest

from oracle import field as F
from oracle import mlp as Mo
from synth import fields as S

pytestmark = pytest.mark.gpu


# ragged extents, a single voxel column, boxes within one block and over
# several, a centre outside the volume, a box that misses it
@pytest.mark.parametrize("dims,n,scales", [((37, 29, 23), 301, (0.2, 1.0)), ((1, 1, 70), 9, (0.3, 2.0)),
                                           ((70, 9, 33), 65, (0.4, 3.0)), ((64, 64, 64), 130, (1.0, 4.0))])
def test_box_moments_direct_and_from_tables(dims, n, scales):
    import torch

    import paper_2608_14112_amd as g
    print(f"feature boxes {dims} n={n}", flush=True)
    p = S.random_params(n, dims, seed=n, scale_range=scales).astype(np.float32)
    p[0, 0] = -2.0
    p[1, 1] = 1e4
    f = np.random.default_rng(n).uniform(0.1, 1.0, size=dims[::-1]).astype(np.float32)
    wide = p[:, :1].copy()
    wide[:3, 0] = [d / 2 for d in dims]
    wide[7:10, 0] = np.log(max(dims) * 16.0)
    ft = torch.from_numpy(f).cuda()
    ctx = g.Context(k=3.0)
    got = []
    for q in (p, np.concatenate([p] + [wide] * 9000, 1)):
        P = g.Params(ctx, q.shape[1]).upload(q)
        got.append(g.features(ctx, P, ft, g.Grid(*dims), 1, 0.3).cpu().numpy()[:n, 13:15])
    ref = Mo.features(f.astype(np.float64), F.Grid(*dims), p.astype(np.float64), 1, 0.3,
                      3.0)[:, 13:15]
    for x in got:
        assert np.allclose(x, ref, rtol=2.5e-7, atol=1e-9)
