"""The seed draws where their two-stage selection can go wrong: volumes of one
voxel along an axis or not a multiple of a block, budgets that take every
eligible voxel or a single one, gradients that are nearly equal, zero almost
everywhere, or near the ends of the float range.  Counts, seeds (through the
jittered centres) and the 99th percentile are exact."""
import numpy as np
import pytest

from oracle import alloc as A
from synth import fields as S

pytestmark = pytest.mark.gpu


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _field(kind, dims, seed):
    rng = np.random.default_rng(seed)
    f = rng.uniform(0.0, 1.0, size=dims[::-1]).astype(np.float32)
    if kind == "ramp":         # equal gradients along x up to rounding
        f = (0.1 + 0.001 * np.arange(dims[0], dtype=np.float32))[None, None, :] + 0 * f
    elif kind == "spot":       # few eligible voxels
        f = np.full(dims[::-1], 0.5, np.float32)
        f[tuple(s // 2 for s in dims[::-1])] = 0.9
    elif kind == "tiny":       # gradients of a few units in the last place
        f = (0.5 + 1e-7 * f).astype(np.float32)
    elif kind == "huge":
        f = (f * np.float32(1e37)).astype(np.float32)
    return np.ascontiguousarray(f.astype(np.float32))


CASES = [("noise", (1, 1, 700), 40), ("noise", (700, 1, 1), 40), ("noise", (1, 90, 70), 300),
         ("noise", (33, 17, 9), 200), ("noise", (64, 64, 33), 1), ("noise", (64, 64, 33), 2),
         ("noise", (50, 41, 37), "all"), ("ramp", (40, 30, 20), 500), ("spot", (40, 30, 20), 10),
         ("tiny", (64, 40, 20), 700), ("huge", (40, 30, 20), 700), ("noise", (130, 127, 65), 9000)]


@pytest.mark.parametrize("kind,dims,budget", CASES)
def test_draws_match_oracle(kind, dims, budget):
    g, torch = _lib()
    f = _field(kind, dims, 5)
    g32 = A.gradient_magnitude32(f)
    occ = f.ravel() > np.float32(A.OCC_THRESHOLD)
    if budget == "all":
        n_el = int((occ & (g32.ravel() > 0)).sum())
        budget = A.max_feasible_budget(n_el, int(occ.sum()))
    print(f"draw {kind} {dims} budget {budget}", flush=True)
    seed = 77
    ctx = g.Context(k=3.0)
    try:
        det, cov, n_el, n_oc = A.draw_seeds(f, g32, budget, seed)
    except A.BudgetInfeasible as e:
        with pytest.raises(g.BudgetInfeasible) as ge:
            g.allocate(ctx, torch.from_numpy(f).cuda(), g.Grid(*dims), budget, seed)
        assert ge.value.shortfall == e.shortfall
        return
    P, info = g.allocate(ctx, torch.from_numpy(f).cuda(), g.Grid(*dims), budget, seed)
    got = P.download()
    assert info["n_eligible"] == n_el and info["n_occupied"] == n_oc
    assert info["n_detail"] == det.size and info["n_coverage"] == cov.size
    a = A.jitter_centers(det, dims[::-1], (0, 0, 0), seed, 0)
    b = A.jitter_centers(cov, dims[::-1], (0, 0, 0), seed, 1)
    assert np.array_equal(got[0:3, :det.size], a)
    assert np.array_equal(got[0:3, det.size:], b)
    assert info["g99"] == float(A.percentile_order_stat(g32.ravel()[occ]))


def test_two_allocations_through_one_context():
    """The second, larger, draws from buffers the first one's binning used."""
    g, torch = _lib()
    ctx = g.Context(k=3.0)
    for dims, budget in (((40, 36, 32), 800), ((96, 90, 70), 5000), ((40, 36, 32), 800)):
        print(f"draw again {dims}", flush=True)
        f = S.spectral_field(dims[::-1], seed=2).numpy()
        det, cov, _, _ = A.draw_seeds(f, A.gradient_magnitude32(f), budget, 3)
        P, _ = g.allocate(ctx, torch.from_numpy(f).cuda(), g.Grid(*dims), budget, 3)
        got = P.download()
        assert np.array_equal(got[0:3, :det.size], A.jitter_centers(det, dims[::-1], (0, 0, 0), 3, 0))
        assert np.array_equal(got[0:3, det.size:], A.jitter_centers(cov, dims[::-1], (0, 0, 0), 3, 1))
