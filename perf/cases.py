"""Timed cases of the encoder: what programs that use it have it do.

Each case is one call (or the calls that a user's loop makes together) through the Python
binding: decoding a primitive set to voxels, gradients for a caller's own optimiser, the
autograd bridge, refinement from the smallest to the largest workload, many volumes at
once, the structure-aware allocation, the warm start and its network's training, and the
paper's sampled loop.

A case is a dict of plain values; `op` names the call.  Fields and primitives are made
here, from the seed alone: fields of tanh level-set fronts of noisy spheres over a
multi-octave background, primitives seeded like an allocation (55 % where the gradient is large, 45 % uniform, each group in voxel
order), with anisotropic random frames whose 3-sigma supports cover each voxel `cover`
times on average, and weights that sum to about the field.
"""
import math
import random

import numpy as np
import torch

import paper_2608_14112_amd as gve
from paper_2608_14112_amd.autograd import GaussianField

DEV = "cuda"
K = 3.0
MLP_FLOPS = 2 * (16 * 128 + 128 * 128 + 128 * 11)  # multiply-adds of one row, forward


# ---- the cases -----------------------------------------------------------------------

def listed():
    return [
        # the smallest decode: 64^3 voxels x 2,048 primitives, where launches and host
        # reads count
        {"name": "decode_64", "op": "evaluate", "nx": 64, "ny": 64, "nz": 64, "n": 2048,
         "cover": 20.0, "origin": 0},
        # decoding a large representation for display or export, ragged and off the origin
        {"name": "decode_509", "op": "evaluate", "nx": 509, "ny": 448, "nz": 391, "n": 200003,
         "cover": 20.0, "origin": 1},
        # the field as a layer of a torch model: forward and backward through autograd
        {"name": "autograd_block", "op": "autograd", "nx": 117, "ny": 96, "nz": 83, "n": 4099,
         "cover": 20.0},
        # loss and gradient with reproducible sums, for a caller's own optimiser
        {"name": "grad_reproducible", "op": "loss_grad", "nx": 250, "ny": 233, "nz": 260,
         "n": 60000, "cover": 20.0, "deterministic": True, "origin": 1},
        # the 64^3 x 2,048 workload: a 20-iteration refinement at lr 1e-3, tuned shape
        {"name": "refine_64", "op": "refine", "nx": 64, "ny": 64, "nz": 64, "n": 2048,
         "cover": 20.0, "iters": 20, "lr": 1e-3, "tuned": True},
        # the 256^3 x 65,536 workload, tuned shape
        {"name": "refine_256", "op": "refine", "nx": 256, "ny": 256, "nz": 256, "n": 65536,
         "cover": 20.0, "iters": 8, "lr": 8e-3, "tuned": True},
        # the paper's scale: 1024^3 x 1.4M with the default options
        {"name": "refine_1024", "op": "refine", "nx": 1024, "ny": 1024, "nz": 1024, "n": 1400000,
         "cover": 20.0, "iters": 2, "lr": 8e-3, "tuned": False},
        # uneven volumes refined together
        {"name": "batch_12", "op": "batch_refine", "items": 12, "lo": 64, "hi": 224,
         "shapes": 7, "density": 1 / 200, "cover": 20.0, "iters": 4, "lr": 8e-3},
        # a new encoding starts here: seeds, frames, scales and weights of 262,144 primitives
        {"name": "allocate_512", "op": "allocate", "nx": 512, "ny": 512, "nz": 512, "n": 262144},
        # the learned correction applied to an allocation, with its loss check
        {"name": "warmstart_384", "op": "warmstart", "nx": 384, "ny": 384, "nz": 384, "n": 110592,
         "cover": 20.0},
        # one epoch of the warm-start network on the pairs of one 512^3 encoding
        {"name": "train_262144", "op": "mlp_train", "rows": 262144, "batch": 4096, "epochs": 1},
        # the paper's sampled loop: an encoding resumed, 100 iterations, and read back
        {"name": "sampled_640", "op": "paper", "nx": 640, "ny": 640, "nz": 640, "n": 400000,
         "iters": 100, "samples": 3072},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _shape(rng, voxels, spread=1.5):
    """Three edges of about `voxels` voxels together, uneven by up to `spread`."""
    e = [math.exp(rng.uniform(-math.log(spread), math.log(spread))) for _ in range(3)]
    f = (voxels / (e[0] * e[1] * e[2])) ** (1 / 3)
    return {a: max(16, int(round(f * x))) for a, x in zip(("nx", "ny", "nz"), e)}


def draw(rng):
    op = rng.choice(["evaluate", "evaluate", "autograd", "loss_grad", "refine", "refine",
                     "batch_refine", "allocate", "warmstart", "mlp_train", "paper"])
    if op == "mlp_train":
        return {"op": op, "rows": int(_log(rng, 8000, 400000)),
                "batch": rng.choice([512, 1000, 2048, 4096, 8192]), "epochs": 1}
    if op == "batch_refine":
        return {"op": op, "items": rng.randint(2, 24), "lo": rng.randint(32, 96),
                "hi": rng.randint(128, 256), "shapes": rng.randint(0, 10 ** 6),
                "density": 1 / _log(rng, 128, 800), "cover": rng.uniform(12, 24),
                "iters": rng.randint(2, 6), "lr": 8e-3}
    span = {"evaluate": (3e4, 1.5e8), "autograd": (3e4, 4e6), "loss_grad": (3e4, 4e7),
            "refine": (3e4, 1.3e8), "allocate": (2.5e5, 2e8), "warmstart": (2.5e5, 8e7),
            "paper": (2e6, 4e8)}[op]
    vox = _log(rng, *span)
    c = {"op": op, **_shape(rng, vox)}
    c["n"] = max(64, int(c["nx"] * c["ny"] * c["nz"] / _log(rng, 128, 800)))
    if op not in ("allocate", "paper"):
        c["cover"] = rng.uniform(12, 24)
    if op in ("evaluate", "loss_grad"):
        c["origin"] = rng.randint(0, 3)
    if op == "loss_grad":
        c["deterministic"] = rng.random() < 0.5
    if op == "refine":
        c["iters"] = rng.randint(2, 20)
        c["lr"] = rng.choice([1e-3, 8e-3])
        c["tuned"] = rng.random() < 0.5
    if op == "paper":
        c["iters"] = rng.randint(20, 120)
        c["samples"] = rng.choice([1024, 3072, 3072, 8192])
    return c


# ---- inputs --------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)


def _rand(gen, *shape):
    return torch.rand(*shape, device=DEV, generator=gen)


def _field(shape, gen):
    """float32 [nz, ny, nx] in [0, 1]: tanh fronts of noisy spheres over a background whose
    octaves follow k^(-1/3) amplitudes."""
    nz, ny, nx = shape
    edge = max(shape)
    out = torch.zeros(shape, device=DEV)
    for octave in range(2, 6):
        m = [max(2, (s * 2 ** octave) // edge + 2) for s in shape]
        r = torch.randn(1, 1, *m, device=DEV, generator=gen) * 2.0 ** (-octave / 3)
        for z0 in range(0, nz, 64):  # slabs: linear in z between the coarse planes
            zs = torch.arange(z0, min(nz, z0 + 64), device=DEV, dtype=torch.float32)
            t = zs * ((m[0] - 1) / max(nz - 1, 1))
            lo = t.floor().clamp(max=m[0] - 2)
            w = (t - lo).view(-1, 1, 1)
            lo = lo.long()
            plane = r[0, 0, lo] * (1 - w) + r[0, 0, lo + 1] * w
            out[z0:z0 + 64] += torch.nn.functional.interpolate(
                plane[:, None], size=(ny, nx), mode="bilinear", align_corners=True)[:, 0]
    lo, hi = out.min(), out.max()
    out.sub_(lo).mul_(0.1 / (hi - lo).clamp_min(1e-12))
    y = torch.arange(ny, device=DEV, dtype=torch.float32).view(1, -1, 1)
    x = torch.arange(nx, device=DEV, dtype=torch.float32).view(1, 1, -1)
    par = _rand(gen, 12, 8).cpu().tolist()
    for z0 in range(0, nz, 64):
        z = torch.arange(z0, min(nz, z0 + 64), device=DEV, dtype=torch.float32).view(-1, 1, 1)
        best = torch.zeros((z.shape[0], ny, nx), device=DEV)
        for p in par:
            c = (p[0] * nx, p[1] * ny, p[2] * nz)
            rad = (0.05 + 0.14 * p[3]) * edge
            wid = (2 + 6 * p[4]) * edge / 1024 + 0.5
            d = torch.sqrt((x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2)
            wob = 0.1 * rad * torch.sin(x * (6.0 / rad) + p[5] * 6) * torch.sin(y * (6.0 / rad) + p[6] * 6)
            best = torch.maximum(best, d.sub_(wob).sub_(rad).mul_(-1.0 / wid).tanh_().add_(1).mul_(0.45))
        out[z0:z0 + 64] += best
    lo, hi = out.min(), out.max()
    return out.sub_(lo).div_((hi - lo).clamp_min(1e-12)).contiguous()


def _seeds(field, n, gen):
    """Voxel index of n seeds: 55 % by gradient magnitude, 45 % uniform, each in voxel order;
    and the 99th percentile of the sampled gradients."""
    nz, ny, nx = field.shape
    M = field.numel()
    f = field.view(-1)
    det = int(0.55 * n + 0.5)
    pool = min(8 * n, 4 * M) + 256
    v = (_rand(gen, pool).double() * M).long().clamp_(max=M - 1)
    x, y, z = v % nx, (v // nx) % ny, v // (nx * ny)
    gm = torch.zeros(pool, device=DEV)
    for c, size, stride in ((x, nx, 1), (y, ny, nx), (z, nz, nx * ny)):
        up, dn = (c < size - 1).long() * stride, (c > 0).long() * stride
        gm += (0.5 * (f[v + up] - f[v - dn])) ** 2
    gm = gm.sqrt_()
    key = -torch.log(_rand(gen, pool).clamp_min(1e-12)) / gm.clamp_min(1e-9)
    a = v[torch.topk(key, det, largest=False).indices].sort().values
    b = (_rand(gen, n - det).double() * M).long().clamp_(max=M - 1).sort().values
    g99 = float(torch.quantile(gm[:1 << 20], 0.99))
    return torch.cat([a, b]), det, g99


def _primitives(field, n, cover, gen, origin=(0, 0, 0)):
    """theta float32 [11, n] (and the detail count and 99th percentile gradient)."""
    nz, ny, nx = field.shape
    M = field.numel()
    v, det, g99 = _seeds(field, n, gen)
    s = (cover * M / (4 / 3 * math.pi * K ** 3 * n)) ** (1 / 3)  # geometric mean scale
    th = torch.empty(11, n, device=DEV)
    for a, c in enumerate((v % nx, (v // nx) % ny, v // (nx * ny))):
        th[a] = c.float() + origin[a] + _rand(gen, n) - 0.5
    q = torch.randn(4, n, device=DEV, generator=gen)
    th[3:7] = q / q.norm(dim=0) * (0.8 + 0.4 * _rand(gen, n))
    th[7:10] = math.log(s) + 0.25 * torch.randn(3, n, device=DEV, generator=gen)
    vol = n / M * (2 * math.pi) ** 1.5 * th[7:10].sum(0).exp()
    th[10] = field.view(-1)[v] / vol * (0.7 + 0.6 * _rand(gen, n))
    return th.contiguous(), det, g99


class _View:
    """A device buffer of the library's, for torch to look at; keeps its owner alive."""

    def __init__(self, owner, ptr, shape):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (ptr, False), "shape": shape, "typestr": "<f4",
                                         "version": 2, "strides": None}


def _theta(params, owner=None):
    """The parameters on the device as a tensor, which holds what owns their memory."""
    view = _View(owner or params, params.device_ptr(), (11, params.n))
    t = torch.as_tensor(view, device=DEV)
    t.owner = view
    return t


def _origin(case):
    return ((0, 0, 0), (-37, 12, 501), (5, -400, 3), (1200, 1200, -64))[case.get("origin", 0)]


def _batch_grids(case):
    rng = random.Random(case["shapes"])
    return [tuple(rng.randint(case["lo"], case["hi"]) for _ in range(3))
            for _ in range(case["items"])]


def _network(ctx, seed):
    """A network whose correction is small and narrows the primitives, which these inputs
    gain from, so that the full correction is taken as with a trained one."""
    mlp = gve.MLP(ctx, seed=seed)
    flat = mlp.export()
    flat[18688:20096] *= 0.0005
    flat[20096 + 7:20096 + 10] = -0.03
    mlp.load(flat)
    return mlp


def prepare(case, seed):
    gen = _gen(seed)
    op = case["op"]
    if op == "mlp_train":
        ctx = gve.Context()
        X = torch.randn(case["rows"], 16, device=DEV, generator=gen)
        T = torch.tanh(X @ torch.randn(16, 11, device=DEV, generator=gen) * 0.5)
        T = T + 0.5 * torch.randn(case["rows"], 11, device=DEV, generator=gen)
        mlp = gve.MLP(ctx, seed=seed & 0xFFFF)
        return {"case": case, "ctx": ctx, "X": X, "T": T.contiguous(), "mlp": mlp,
                "start": mlp.export(), "seed": seed & 0xFFFF}
    if op == "batch_refine":
        grids = [gve.Grid(*s) for s in _batch_grids(case)]
        fields, thetas = [], []
        for g in grids:
            f = _field(g.shape, gen)
            n = max(64, int(f.numel() * case["density"]))
            thetas.append(_primitives(f, n, case["cover"], gen)[0])
            fields.append(f.view(-1))
        ctx = gve.Context(lr=case["lr"], ell_min=math.log(0.25),
                          ell_max=math.log(max(2.0, case["hi"] / 16)))
        batch = gve.Batch(ctx, grids, [t.shape[1] for t in thetas])
        return {"case": case, "ctx": ctx, "batch": batch, "fields": torch.cat(fields),
                "start": torch.cat(thetas, 1).contiguous(), "theta": _theta(batch.params, batch)}
    shape = (case["nz"], case["ny"], case["nx"])
    org = _origin(case)
    grid = gve.Grid(case["nx"], case["ny"], case["nz"], *org)
    field = _field(shape, gen)
    state = {"case": case, "grid": grid, "field": field, "seed": seed & 0xFFFF}
    if op == "allocate":
        return {**state, "ctx": gve.Context()}
    n = case["n"]
    if op == "paper":
        th, _, _ = _primitives(field, n, 8.0, gen)
        th12 = torch.cat([th[:10], field.view(-1)[_voxel_of(th, shape)][None],
                          torch.full((1, n), math.log(0.1 / 0.9), device=DEV)])
        ctx = gve.Context(k=5.0)
        opts = gve.paper_options(samples=case["samples"], ell_hi=math.log(max(shape) / 16))
        return {**state, "ctx": ctx, "opts": opts, "params": gve.PaperParams(ctx, n),
                "start": th12.cpu().numpy()}
    th, det, g99 = _primitives(field, n, case["cover"], gen, org)
    state["start"] = th
    if op == "autograd":
        up = torch.randn(shape, device=DEV, generator=gen)
        return {**state, "layer": GaussianField(n, grid, k=K), "up": up,
                "leaf": th.clone().requires_grad_(True)}
    edge = max(shape)
    opt = {"ell_min": math.log(0.25), "ell_max": math.log(max(2.0, edge / 16))}
    if op == "refine":
        opt["lr"] = case["lr"]
        if case["tuned"]:
            opt["brick"] = 0
    ctx = gve.Context(k=K, deterministic=bool(case.get("deterministic", False)), **opt)
    params = gve.Params(ctx, n).upload_device(th)
    state.update(ctx=ctx, params=params, theta=_theta(params))
    if op == "refine" and case["tuned"]:
        gve.autotune(ctx, field, params=params, grid=grid)
    if op == "evaluate":
        state["out"] = torch.empty(shape, device=DEV)
    if op == "loss_grad":
        state["grad"] = torch.empty(11, n, device=DEV)
    if op == "warmstart":
        state.update(mlp=_network(ctx, seed & 0xFFFF), det=det, g99=g99)
    return state


def _voxel_of(th, shape):
    nz, ny, nx = shape
    c = [(th[a] + 0.5).floor().long().clamp_(0, s - 1) for a, s in enumerate((nx, ny, nz))]
    return c[0] + nx * (c[1] + ny * c[2])


# ---- one pass ------------------------------------------------------------------------

def run(state):
    case = state["case"]
    op = case["op"]
    if op == "evaluate":
        return gve.evaluate(state["ctx"], state["params"], state["grid"], state["out"])
    if op == "autograd":
        leaf = state["leaf"]
        leaf.grad = None
        v = state["layer"](leaf)
        v.backward(state["up"])
        return v.detach(), leaf.grad
    if op == "loss_grad":
        loss = gve.loss_grad(state["ctx"], state["params"], state["field"], state["grid"],
                             state["grad"])
        return loss, state["grad"]
    if op == "refine":
        state["params"].upload_device(state["start"])
        losses = gve.refine(state["ctx"], state["params"], state["field"], state["grid"],
                            case["iters"])
        return losses.astype(np.float32), state["theta"]
    if op == "batch_refine":
        state["batch"].params.upload_device(state["start"])
        losses = gve.batch_refine(state["ctx"], state["batch"], state["fields"], case["iters"])
        return losses.astype(np.float32), state["theta"]
    if op == "allocate":
        params, info = gve.allocate(state["ctx"], state["field"], state["grid"], case["n"],
                                    state["seed"])
        return _theta(params), {k: info[k] for k in sorted(info)}
    if op == "warmstart":
        state["params"].upload_device(state["start"])
        applied, losses = gve.warmstart(state["ctx"], state["mlp"], state["params"],
                                        state["field"], state["grid"], state["det"],
                                        state["g99"])
        return int(applied), losses.astype(np.float32), state["theta"]
    if op == "mlp_train":
        state["mlp"].load(state["start"])
        losses = gve.mlp_train(state["ctx"], state["mlp"], state["X"], state["T"],
                               case["epochs"], batch=case["batch"], seed=state["seed"])
        return losses.astype(np.float32), state["mlp"].export()
    if op == "paper":
        state["params"].upload(state["start"])
        losses = gve.paper_refine(state["ctx"], state["params"], state["field"], state["grid"],
                                  state["opts"], state["seed"], case["iters"],
                                  schedule_len=1500)
        return losses.astype(np.float32), state["params"].download()
    raise ValueError(op)


# ---- what a pass cannot do without ---------------------------------------------------

def work(case):
    """Each input read once, each output written once; 20 operations per in-support
    (primitive, voxel) pair forward, 58 with the gradient, pairs from the mean coverage."""
    op = case["op"]
    if op == "mlp_train":
        rows = case["rows"] * case["epochs"]
        return {"bytes": 4 * 27 * rows + 12 * 20107, "flops": 3 * MLP_FLOPS * rows}
    if op == "batch_refine":
        M = sum(a * b * c for a, b, c in _batch_grids(case))
        n = M * case["density"]
        it = case["iters"]
        return {"bytes": it * (4 * M + 6 * 44 * n), "flops": it * 58 * case["cover"] * M}
    M, n = case["nx"] * case["ny"] * case["nz"], case["n"]
    if op == "paper":
        # parameters and moments read and written; the volume only at the samples and centres
        return {"bytes": case["iters"] * (288 * n + 32 * n) + 96 * n + 4 * M,
                "flops": case["iters"] * 200 * n}
    if op == "allocate":
        return {"bytes": 4 * M + 44 * n, "flops": 20 * M + 20 * 10 * M}
    P = case["cover"] * M
    if op == "evaluate":
        return {"bytes": 44 * n + 4 * M, "flops": 20 * P}
    if op == "autograd":
        return {"bytes": 88 * n + 8 * M, "flops": 58 * P}
    if op == "loss_grad":
        return {"bytes": 88 * n + 4 * M, "flops": 58 * P}
    if op == "refine":
        it = case["iters"]
        return {"bytes": it * (4 * M + 6 * 44 * n), "flops": it * 58 * P}
    if op == "warmstart":
        return {"bytes": 4 * M + 88 * n, "flops": 2 * 20 * P + MLP_FLOPS * n}
    raise ValueError(op)


# ---- 64-bit values -------------------------------------------------------------------

def _chunk_field(th, xyz, k):
    """Truncated contributions [chunk, M] of a few primitives at every voxel, float64."""
    mu, q, l, c = th[0:3], th[3:7], th[7:10], th[10]
    q = q / q.norm(dim=0)
    w, x, y, z = q
    R = torch.stack([
        torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)]),
        torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)]),
        torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])])
    m2 = 0.0
    for j in range(3):
        t = sum(R[a, j][:, None] * (xyz[a][None] - mu[a][:, None]) for a in range(3))
        m2 = m2 + (t * torch.exp(-l[j])[:, None]) ** 2
    g = torch.where(m2 < k * k, torch.exp(-0.5 * m2), torch.zeros((), device=DEV,
                                                                dtype=torch.float64))
    return c[:, None] * g


def exact(case, seed):
    """The truncated sum and its gradient over every (primitive, voxel) pair in float64, for
    the sizes where that takes seconds."""
    op = case["op"]
    if op not in ("evaluate", "autograd", "loss_grad"):
        return None
    M, n = case["nx"] * case["ny"] * case["nz"], case["n"]
    if M * n > (1.2e10 if op == "evaluate" else 5e9):
        return None
    gen = _gen(seed)
    shape = (case["nz"], case["ny"], case["nx"])
    org = _origin(case)
    field = _field(shape, gen)
    th = _primitives(field, n, case["cover"], gen, org)[0].double()
    ax = [torch.arange(s, device=DEV, dtype=torch.float64) + o
          for s, o in zip((case["nx"], case["ny"], case["nz"]), org)]
    zz, yy, xx = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    xyz = [xx.reshape(-1), yy.reshape(-1), zz.reshape(-1)]
    step = max(1, int(6e7 // M))
    V = torch.zeros(M, device=DEV, dtype=torch.float64)
    for i in range(0, n, step):
        V += _chunk_field(th[:, i:i + step], xyz, K).sum(0)
    if op == "evaluate":
        return V.view(shape)
    if op == "autograd":
        up = torch.randn(shape, device=DEV, generator=gen).double().view(-1)
    else:
        r = V - field.double().view(-1)
        up = 2 * r
    grad = torch.empty_like(th)
    for i in range(0, n, step):
        t = th[:, i:i + step].clone().requires_grad_(True)
        (_chunk_field(t, xyz, K).sum(0) @ up).backward()
        grad[:, i:i + step] = t.grad
    if op == "autograd":
        return V.view(shape), grad
    return float(r.square().sum()), grad
