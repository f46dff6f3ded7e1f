"""The sampled loop's batching: points bucketed by one workgroup (up to 16,384)
or by the radix sort beyond, iterations sampled together against one at a time,
and primitives on both sides of the list of reached points.

Accumulators are float64 sums in any order, so the float32 values formed from
them agree to a rounding of the last place (2^-23, doubled for the quotient);
gradients and objective follow the tolerances of the oracle comparison.
"""
import math

import numpy as np
import pytest

from oracle import field as F
from oracle import paper as Pp
from synth import fields as S
from tests.parity import check_grad

pytestmark = pytest.mark.gpu

GRID = F.Grid(40, 36, 30, 2, -3, 1)


def _lib():
    import torch

    import paper_2608_14112_amd as g
    assert torch.cuda.is_available()
    return g, torch


def _field():
    gen = S.random_params(60, (40, 36, 30), seed=31, scale_range=(2.0, 5.0), weight_range=(0.2, 1.0))
    f = S.mixture_field(gen, GRID.shape)
    return ((f - f.min()) / (f.max() - f.min())).astype(np.float32)


def _theta(n, seed, sr):
    p = S.random_params(n, (40, 36, 30), seed=seed, scale_range=sr, unit_quat=False)
    rng = np.random.default_rng(seed + 1)
    th = np.zeros((12, n))
    th[0:10] = p[0:10]
    th[0] += GRID.x0
    th[1] += GRID.y0
    th[2] += GRID.z0
    th[10] = rng.uniform(0.0, 1.0, n)
    th[11] = rng.normal(0.0, 0.5, n)
    return th.astype(np.float32)


def _gg(g):
    return g.Grid(GRID.nx, GRID.ny, GRID.nz, GRID.x0, GRID.y0, GRID.z0)


@pytest.mark.parametrize("cell", [4.0, 64.0])
@pytest.mark.parametrize("npts", [1, 8192, 8193, 16384, 16385])
def test_evaluation_does_not_depend_on_how_points_are_bucketed(npts, cell):
    """All points in one call against calls of 5,000 (cell 64: one cell)."""
    g, torch = _lib()
    print(f"paper_eval {npts} points cell {cell}", flush=True)
    ctx = g.Context()
    P = g.PaperParams(ctx, 90).upload(_theta(90, 5, (1.5, 4.0)))
    o = g.paper_options(cell=cell)
    rng = np.random.default_rng(npts)
    pts = torch.from_numpy((rng.uniform(-6, 46, size=(npts, 3))).astype(np.float32)).cuda()
    vt, den = g.paper_eval(ctx, P, _gg(g), o, pts)
    for a in range(0, npts, 5000):
        v2, d2 = g.paper_eval(ctx, P, _gg(g), o, pts[a:a + 5000].contiguous())
        assert torch.allclose(vt[a:a + 5000], v2, rtol=2.4e-7, atol=1e-12)
        assert torch.allclose(den[a:a + 5000], d2, rtol=1.2e-7, atol=1e-12)


@pytest.mark.parametrize("samples", [50, 4096, 4097, 8193])
def test_batched_iterations_equal_single_ones(samples):
    """40 iterations in one call (batches of 32 and 8, or singly past 8,192
    samples) against 40 calls of one.  Learning rate 0 keeps the parameters, so
    every objective must agree."""
    g, torch = _lib()
    print(f"paper_refine samples {samples}", flush=True)
    ctx = g.Context()
    f = torch.from_numpy(_field()).cuda()
    th = _theta(80, 9, (1.5, 4.0))
    o = g.paper_options(samples=samples, lr=0.0, cell=8.0)
    P = g.PaperParams(ctx, 80).upload(th)
    a = g.paper_refine(ctx, P, f, _gg(g), o, seed=4, iters=40, schedule_len=60)
    assert np.array_equal(P.download(), th)
    b = [g.paper_refine(ctx, P, f, _gg(g), o, seed=4, iters=1, first_iter=i, schedule_len=60)[0]
         for i in range(40)]
    assert np.allclose(a, b, rtol=1e-12)


def test_few_points_per_primitive_match_oracle():
    """Narrow primitives: most reach 0 to 8 points (the kept list), some more."""
    g, torch = _lib()
    f = _field()
    th = _theta(300, 17, (0.25, 1.1)).astype(np.float64)
    base = dict(k=5.0, samples=400, lam_rho=0.2, lam_sm_start=0.15, lam_sm_end=0.05, lam_anc=0.05,
                lam_aniso=0.5, lam_cap=0.5, ell_lo=math.log(0.3), ell_hi=math.log(3.5), cell=8.0)
    o = g.paper_options(**base)
    po = Pp.Options(k=o.k, rho0=o.rho0, samples=o.samples, frac_hi=o.frac_hi, frac_mid=o.frac_mid,
                    v_hi=o.v_hi, v_occ=o.v_occ, lam_rho=o.lam_rho, lam_sm=o.lam_sm_start,
                    lam_anc=o.lam_anc, lam_aniso=o.lam_aniso, lam_cap=o.lam_cap,
                    aniso_max=o.aniso_max, ell_lo=o.ell_lo, ell_hi=o.ell_hi)
    rp, rq, rv = Pp.sample_points(f, GRID, o.samples, seed=12, it=0, opt=po)
    pts = np.concatenate([rp, rq]).astype(np.float32)
    vals = rv.astype(np.float32)
    p64, v64 = pts.astype(np.float64), vals.astype(np.float64)
    reached = (Pp.kernels(th, p64, po.k) > 0).sum(axis=1)
    assert np.count_nonzero((reached > 0) & (reached <= 8)) > 50
    assert np.count_nonzero(reached > 8) > 5 and np.count_nonzero(reached == 0) > 5
    ctx = g.Context()
    P = g.PaperParams(ctx, 300).upload(th.astype(np.float32))
    print("paper_loss_grad narrow primitives", flush=True)
    L, parts, grad = g.paper_loss_grad(ctx, P, torch.from_numpy(f).cuda(), _gg(g), o,
                                       o.lam_sm_start, torch.from_numpy(pts).cuda(),
                                       torch.from_numpy(vals).cuda())
    n = o.samples
    Lr, pr = Pp.objective(th, f, GRID, p64[:n], p64[n:], v64, po)
    assert abs(L - Lr) <= 1e-5 * Lr, (parts, pr)
    gr = Pp.objective_grad(th, f, GRID, p64[:n], p64[n:], v64, po)
    got = grad.cpu().numpy().astype(np.float64)
    check_grad(got[0:11], gr[0:11])
    assert np.linalg.norm(got[11] - gr[11]) <= 1e-3 * np.linalg.norm(gr[11])
