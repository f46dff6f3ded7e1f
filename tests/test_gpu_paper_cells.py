"""The sampled loop with many cells.  The cell size decides how points are bucketed
(a workgroup per iteration, or the radix sort and chip-wide ranges) and which
cells a primitive visits, not which points it reaches: objectives and evaluations
are those of the default cell of 32 up to the order of float64 sums (1e3 terms of
1.1e-16, and up to 1e3 more where a residual cancels: 1e-10)."""
import math

import numpy as np
import pytest

from synth import fields as S

pytestmark = pytest.mark.gpu

DIMS = (120, 100, 90)


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _theta(n):
    p = S.random_params(n, DIMS, seed=3, scale_range=(0.8, 3.0), unit_quat=False)
    rng = np.random.default_rng(4)
    th = np.zeros((12, n), np.float32)
    th[0:10] = p[0:10]
    th[10] = rng.uniform(0.0, 1.0, n)
    th[11] = rng.normal(0.0, 0.5, n)
    return th


# cells: 90, 4,050, 16,875, 135,000, 630,000 and 1,080,000; 20 iterations in
# batches of 20 down to 14, and 3
@pytest.mark.parametrize("samples", [200, 5000])
@pytest.mark.parametrize("iters", [20, 3])
def test_objective_does_not_depend_on_the_cell(samples, iters):
    g, torch = _lib()
    rng = np.random.default_rng(5)
    f = torch.from_numpy(rng.uniform(size=DIMS[::-1]).astype(np.float32)).cuda()
    ref = None
    for cell in (32.0, 6.0, 4.0, 2.0, 1.2, 1.0):
        print(f"paper cells samples={samples} iters={iters} cell={cell}", flush=True)
        ctx = g.Context()
        o = g.paper_options(samples=samples, lr=0.0, cell=cell, ell_hi=math.log(8.0))
        P = g.PaperParams(ctx, 500).upload(_theta(500))
        h = g.paper_refine(ctx, P, f, g.Grid(*DIMS), o, seed=6, iters=iters, schedule_len=60)
        ref = h if ref is None else ref
        assert np.allclose(h, ref, rtol=1e-10)


@pytest.mark.parametrize("npts", [100, 8192, 8193])
def test_evaluation_does_not_depend_on_the_cell(npts):
    g, torch = _lib()
    rng = np.random.default_rng(npts)
    pts = torch.from_numpy((rng.uniform(-3, 123, size=(npts, 3))).astype(np.float32)).cuda()
    ctx = g.Context()
    P = g.PaperParams(ctx, 500).upload(_theta(500))
    ref = None
    # 32,768 cells and one layer more are the two sides of the rule for one set
    for cell, grid in ((32.0, g.Grid(*DIMS)), (1.0, g.Grid(*DIMS)), (1.0, g.Grid(32, 32, 32)),
                       (1.0, g.Grid(32, 32, 33))):
        print(f"paper cells eval {npts} cell={cell} grid {grid.nz}", flush=True)
        vt, den = g.paper_eval(ctx, P, grid, g.paper_options(cell=cell), pts)
        ref = (vt, den) if ref is None else ref
        assert torch.allclose(vt, ref[0], rtol=2.4e-7, atol=1e-12)
        assert torch.allclose(den, ref[1], rtol=1.2e-7, atol=1e-12)
