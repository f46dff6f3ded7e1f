"""Seed draws of fields at the top of the float range: gradients past 2^126, whose
reciprocal is subnormal, some of them infinite (one-sided differences at the
faces).  Counts, seeds and the 99th percentile are exact."""
import numpy as np
import pytest

from oracle import alloc as A

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("top", [3.2e38, 1.2e38, 1e38])
@pytest.mark.parametrize("budget", [20, 700, 6000])
def test_gradients_past_the_reciprocal(top, budget):
    _check(np.random.default_rng(9).uniform(0.02, 1.0, size=(20, 30, 40)).astype(np.float32)
           * np.float32(top), budget, f"top {top}")


def _check(f, budget, name):
    import torch

    import paper_2608_14112_amd as g
    print(f"draw {name} budget {budget}", flush=True)
    dims = f.shape[::-1]
    with np.errstate(over="ignore"):
        g32 = A.gradient_magnitude32(f)
        det, cov, n_el, n_oc = A.draw_seeds(f, g32, budget, 78)
    P, info = g.allocate(g.Context(k=3.0), torch.from_numpy(f).cuda(), g.Grid(*dims), budget, 78)
    got = P.download()
    assert info["n_eligible"] == n_el and info["n_occupied"] == n_oc
    assert np.array_equal(got[0:3, :det.size], A.jitter_centers(det, f.shape, (0, 0, 0), 78, 0))
    assert np.array_equal(got[0:3, det.size:], A.jitter_centers(cov, f.shape, (0, 0, 0), 78, 1))
    occ = f.ravel() > np.float32(A.OCC_THRESHOLD)
    assert info["g99"] == float(A.percentile_order_stat(g32.ravel()[occ]))
