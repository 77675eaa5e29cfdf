"""The work that the performance of this framework is measured on.

Each case is one call (or one whole solve) through the public binding of
``paper_2403_03571_amd``, over the ranges that the repository's workloads,
tests and benchmark use:

* ``eval``     one evaluation of the dual objective with gradient, counts and
               centroids (what every step of a fit or of a Lloyd loop costs);
* ``assign``   the label image of a diagram (Algorithm 1);
* ``fit``      a whole fit of the weights from zero to 1 % (Algorithm 2);
* ``batch``    many uneven 2D fits in one batched solve;
* ``train``    loss and gradient of the warm-start network on a minibatch;
* ``predict``  warm-start weights of one problem (features and inference).

``prepare`` makes what a program holds before the call: the problem's device
arrays, a context with its options, the network.  Weights of the ``eval`` and
``assign`` cases are the costs at the radii of balls of the target volumes (the
squared radii for the squared norm), a user's usual first guess and of the
size of fitted weights.
"""
import math

import numpy as np
import torch

import paper_2403_03571_amd as apd

FEAT, HID, NEIGH = 20, 128, 16


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest problem: a thumbnail with a handful of grains, where
        # launches and the host's part of a call count
        {"name": "eval_2d_smallest", "kind": "eval", "g0": 256, "g1": 256, "g2": 0, "n": 16,
         "prec": "fp32", "lists": True, "mass": False, "power": 2},
        # one evaluation of an EBSD-sized 2D map on the bf16 tier
        {"name": "eval_2d_bf16", "kind": "eval", "g0": 1024, "g1": 1024, "g2": 0, "n": 1000,
         "prec": "bf16", "lists": True, "mass": False, "power": 2},
        # one evaluation of the 3D polycrystal, default options
        {"name": "eval_3d", "kind": "eval", "g0": 256, "g1": 256, "g2": 256, "n": 10000,
         "prec": "fp32", "lists": True, "mass": False, "power": 2},
        # the benchmark's headline: every pixel against every seed, 3D and 2D
        {"name": "eval_3d_every_seed", "kind": "eval", "g0": 256, "g1": 256, "g2": 256, "n": 10000,
         "prec": "fp32", "lists": False, "mass": False, "power": 2},
        {"name": "eval_2d_every_seed", "kind": "eval", "g0": 1024, "g1": 1024, "g2": 0, "n": 1000,
         "prec": "fp32", "lists": False, "mass": False, "power": 2},
        # labels of a ragged 3D volume for rendering or meshing
        {"name": "assign_3d_ragged", "kind": "assign", "g0": 181, "g1": 203, "g2": 97, "n": 3001,
         "prec": "fp32", "lists": True},
        # the double-precision tier, which the paper runs throughout
        {"name": "eval_2d_fp64", "kind": "eval", "g0": 512, "g1": 512, "g2": 0, "n": 500,
         "prec": "fp64", "lists": True, "mass": False, "power": 2},
        # whole fits: the 2D map, the 3D polycrystal, and a batch of 2D maps
        {"name": "fit_2d", "kind": "fit", "g0": 1024, "g1": 1024, "g2": 0, "n": 1000},
        {"name": "fit_3d", "kind": "fit", "g0": 256, "g1": 256, "g2": 256, "n": 10000},
        {"name": "fit_batch_2d", "kind": "batch", "count": 512, "nmin": 50, "nmax": 2000},
        # the warm start: one training minibatch, and a prediction
        {"name": "warm_start_train", "kind": "train", "samples": 4096},
        {"name": "warm_start_predict", "kind": "predict", "g0": 512, "g1": 512, "g2": 0, "n": 700},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, dim, pixels):
    """An uneven grid of about `pixels` pixels (at least 16 along each axis)."""
    side = pixels ** (1.0 / dim)
    r = [math.exp(rng.uniform(-0.3, 0.3)) for _ in range(dim)]
    m = math.exp(sum(math.log(t) for t in r) / dim)
    g = [max(16, int(side * t / m)) for t in r]
    return g + [0] * (3 - dim)


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "assign", "fit", "batch", "train", "predict"])
    dim = rng.choice([2, 3])
    if kind == "train":
        return {"kind": kind, "samples": _log_int(rng, 100, 8192)}
    if kind == "batch":
        lo = _log_int(rng, 50, 300)
        return {"kind": kind, "count": _log_int(rng, 8, 128), "nmin": lo, "nmax": _log_int(rng, lo + 20, 2000)}
    if kind == "predict":
        n = _log_int(rng, 50, 2000)
        g = _grid(rng, 2, n * rng.uniform(300.0, 800.0))
        return {"kind": kind, "g0": g[0], "g1": g[1], "g2": 0, "n": n}
    if kind == "fit":
        # enough pixels per cell that 1 % can be reached (eq. (2.10))
        n = _log_int(rng, 16, 3000) if dim == 2 else _log_int(rng, 30, 4000)
        g = _grid(rng, dim, max(n, 40) * rng.uniform(1200.0, 2000.0))
        return {"kind": kind, "g0": g[0], "g1": g[1], "g2": g[2], "n": n}
    n = _log_int(rng, 16, 10000)
    g = _grid(rng, dim, min(16.0e6, max(65536.0, n * rng.uniform(300.0, 1700.0))))
    if kind == "assign":
        return {"kind": kind, "g0": g[0], "g1": g[1], "g2": g[2], "n": n,
                "prec": rng.choice(["fp32", "fp32", "fp32", "bf16"]), "lists": True}
    prec = rng.choice(["fp32", "fp32", "fp32", "bf16", "fp64"])
    power = 2
    if prec == "fp64":  # the tier over every pair: problems of its usual size
        n = _log_int(rng, 16, 1000)
        g = _grid(rng, dim, max(65536.0, min(1048576.0, n * rng.uniform(300.0, 1000.0))))
        power = rng.choice([2, 2, 1, 3, 4])
    return {"kind": kind, "g0": g[0], "g1": g[1], "g2": g[2], "n": n, "prec": prec,
            "lists": rng.random() < 0.7, "mass": rng.random() < 0.2, "power": power}


# ----------------------------------------------------------------- inputs

def _dim(case):
    return 3 if case["g2"] else 2


def _rotations3(rng, n):
    q = rng.standard_normal((n, 4))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    w, x, y, z = q.T
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                  2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                  2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], axis=1)
    return R.reshape(n, 3, 3)


def _instance(rng, dim, grid, n, sigma, mass=False):
    """Uniform seeds in the unit box, unit-determinant anisotropy, log-normal
    (sigma > 0) or equal target volumes; optionally a ball-shaped domain given
    by pixel weights."""
    x = rng.random((n, dim))
    if dim == 2:
        a, t = rng.uniform(1.0, 3.0, n), rng.uniform(0.0, np.pi, n)
        c, s = np.cos(t), np.sin(t)
        R = np.stack([c, -s, s, c], axis=1).reshape(n, 2, 2)
        ev = np.stack([a, 1.0 / a], axis=1)
    else:
        R = _rotations3(rng, n)
        la = 0.3 * rng.standard_normal((n, 3))
        ev = np.exp(la - la.mean(axis=1, keepdims=True))
    A = (R * ev[:, None, :]) @ R.transpose(0, 2, 1)
    A = 0.5 * (A + A.transpose(0, 2, 1))
    q = None
    omega = 1.0
    if mass:
        r2 = 0.0
        for d in range(dim):
            k = (np.arange(grid[d]) + 0.5) / grid[d] - 0.5
            r2 = r2 + (k * k).reshape([-1 if e == d else 1 for e in range(dim)])
        # full inside radius 0.45, fading to zero over two hundredths
        q = np.rint(255.0 * np.clip((0.46 - np.sqrt(r2)) / 0.02, 0.0, 1.0)).astype(np.uint8).reshape(-1)
        omega = float(q.astype(np.int64).sum()) / 255.0 / float(np.prod(grid))
    v = np.exp(sigma * rng.standard_normal(n)) if sigma > 0.0 else np.ones(n)
    v = v / v.sum() * omega
    v[np.argmax(v)] += omega - v.sum()
    return x, A, v, q


def _weights(dim, v, power=2):
    r = np.sqrt(v / math.pi) if dim == 2 else np.cbrt(0.75 * v / math.pi)
    w = r ** power
    return w - w.mean()


def _dev(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _grid_of(case):
    return (case["g0"], case["g1"], case["g2"])[:_dim(case)]


def _host(case, seed):
    """The case's problem as host arrays: (x, A, v, q, w)."""
    rng = np.random.default_rng(seed)
    dim = _dim(case)
    sigma = 0.0 if case["kind"] == "predict" else 0.3
    x, A, v, q = _instance(rng, dim, _grid_of(case), case["n"], sigma, case.get("mass", False))
    return x, A, v, q, _weights(dim, v, case.get("power", 2))


def _net(seed):
    """He-uniform parameters of the warm-start network (biases small)."""
    rng = np.random.default_rng(seed + 7)
    parts = []
    for i, o in ((FEAT, HID), (HID, HID), (HID, HID), (HID, 1)):
        lim = math.sqrt(6.0 / i)
        parts += [rng.uniform(-lim, lim, i * o), rng.uniform(-0.05, 0.05, o)]
    return np.concatenate(parts).astype(np.float32)


def _samples(case, seed):
    """Training samples with the spread of the features and targets."""
    rng = np.random.default_rng(seed)
    F = rng.standard_normal((case["samples"], FEAT)).astype(np.float32)
    t = (0.3 * rng.standard_normal(case["samples"])).astype(np.float32)
    return F, t


def _batch(case, seed):
    """Uneven 2D maps: side clamp(64 ceil(20 sqrt(n) / 64), 256, 1024).  The
    sizes belong to the case, the maps to the seed."""
    rng = np.random.default_rng(seed)
    sizes = np.random.default_rng([case["count"], case["nmin"], case["nmax"]])
    out = []
    for _ in range(case["count"]):
        n = int(sizes.integers(case["nmin"], case["nmax"] + 1))
        side = int(min(max(64 * math.ceil(20.0 * math.sqrt(n) / 64.0), 256), 1024))
        x, A, v, _ = _instance(rng, 2, (side, side), n, 0.0)
        out.append(((side, side), x, A, v))
    return out


def _problem(grid, x, A, v, q=None, power=2):
    dim = x.shape[1]
    return apd.Problem(dim, grid, (0.0,) * dim, (1.0,) * dim, _dev(x), _dev(A), _dev(v),
                       None if q is None else _dev(q, torch.uint8), power)


def prepare(case, seed):
    kind = case["kind"]
    ctx = apd.Context(torch.cuda.current_device())
    st = {"case": case, "ctx": ctx}
    if kind == "train":
        F, t = _samples(case, seed)
        st.update(net=apd.WarmStart(ctx, _net(seed)), F=_dev(F, torch.float32), t=_dev(t, torch.float32))
    elif kind == "batch":
        st["probs"] = [_problem(*p) for p in _batch(case, seed)]
    else:
        x, A, v, q, w = _host(case, seed)
        st["prob"] = _problem(_grid_of(case), x, A, v, q, case.get("power", 2))
        st["w"] = _dev(w)
        if kind == "predict":
            st["net"] = apd.WarmStart(ctx, _net(seed))
        if not case.get("lists", True):
            ctx.apd_set_culling(False)
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "eval":
        return ctx.apd_dual_objective_grad(st["prob"], st["w"], prec=case["prec"], counts=True, centroids=True)
    if kind == "assign":
        return ctx.apd_assign(st["prob"], st["w"], prec=case["prec"])
    if kind == "fit":
        w, rep = ctx.apd_fit_weights(st["prob"], eps=0.01, max_evals=600)
        return {"w": w, "g": rep.g, "maxrel": rep.max_rel_err, "evals": rep.evals}
    if kind == "batch":
        ws, reps, _ = ctx.apd_fit_weights_batched(st["probs"], eps=0.01, max_evals=600)
        return {"w": torch.cat(ws), "evals": np.array([r.evals for r in reps])}
    if kind == "train":
        loss, grad = st["net"].loss_grad(st["F"], st["t"])
        return {"loss": loss, "grad": grad}
    return st["net"].predict(st["prob"])


# ------------------------------------------------------------------- work

def work(case):
    kind = case["kind"]
    if kind == "train":
        s, p = case["samples"], FEAT * HID + 2 * HID * HID + HID
        # forward and both backward products of every layer (the first layer
        # needs no gradient of its inputs)
        return {"bytes": 4.0 * (s * (FEAT + 1) + 2 * p), "flops": 2.0 * s * (3 * p - FEAT * HID)}
    if kind == "batch":
        n = 0.5 * (case["nmin"] + case["nmax"])
        pix = min(max(400.0 * n, 65536.0), 1048576.0)
        # a fit needs of the order of a hundred evaluations
        return {"bytes": 100.0 * case["count"] * n * 72.0, "flops": 100.0 * case["count"] * pix * 24.0}
    dim, n = _dim(case), case["n"]
    pix = float(np.prod([float(g) for g in _grid_of(case)]))
    seeds = 8.0 * n * (dim + dim * dim + 2)
    # a pixel's cost of one seed: the expanded quadratic form
    form = 12.0 if dim == 2 else 20.0
    if kind == "eval":
        # over every seed each pair needs two fused multiply-adds and a
        # minimum; with lists a pixel needs its own cell and one rival; the
        # double tier evaluates the form for every pair
        flops = (form * n * pix if case["prec"] == "fp64" else 2.0 * form * pix if case["lists"] else 5.0 * n * pix)
        return {"bytes": seeds + 8.0 * n * (2 + dim) + (pix if case["mass"] else 0.0), "flops": flops}
    if kind == "assign":
        return {"bytes": seeds + 4.0 * pix, "flops": 2.0 * form * pix}
    if kind == "fit":
        return {"bytes": 100.0 * (seeds + 8.0 * n), "flops": 100.0 * 2.0 * form * pix}
    layers = FEAT * HID + 2 * HID * HID + HID
    return {"bytes": seeds + 8.0 * n + 4.0 * layers,
            "flops": 2.0 * form * pix + 2.0 * n * layers + 8.0 * n * n}


# ---------------------------------------------------------- 64-bit results

def _assign64(grid, x, A, w, power):
    """Least cost and its seed at every pixel, in double, by chunks: the
    squared norms as a product of monomials of the pixel (about the box
    centre) with each seed's coefficients."""
    dim, dev = x.shape[1], x.device
    e = x - 0.5
    Ae = torch.einsum("nij,nj->ni", A, e)
    pairs = [(r, c) for r in range(dim) for c in range(r, dim)]
    cols = [A[:, r, c] * (1.0 if r == c else 2.0) for r, c in pairs]
    cols += [-2.0 * Ae[:, d] for d in range(dim)] + [(e * Ae).sum(1)]
    if power == 2:
        cols[-1] = cols[-1] - w
    coef = torch.stack(cols)
    J = int(np.prod(grid))
    step = max(1, min(J, (1 << 28) // x.shape[0]))
    lab = torch.empty(J, dtype=torch.int64, device=dev)
    cost = torch.empty(J, dtype=torch.float64, device=dev)
    for j0 in range(0, J, step):
        j = torch.arange(j0, min(J, j0 + step), device=dev)
        k, rest = [], j
        for d in reversed(range(dim)):
            k.insert(0, rest % grid[d])
            rest = rest // grid[d]
        u = [(k[d].double() + 0.5) / grid[d] - 0.5 for d in range(dim)]
        feat = torch.stack([u[r] * u[c] for r, c in pairs] + u + [torch.ones_like(u[0])], dim=1)
        c = feat @ coef
        if power != 2:
            c = c.clamp_min(0.0).pow(0.5 * power) - w
        m = c.min(dim=1)
        cost[j0:j0 + step], lab[j0:j0 + step] = m.values, m.indices
    return lab, cost


def _evaluate64(grid, x, A, v, q, w, power):
    dim, n, dev = x.shape[1], x.shape[0], x.device
    lab, cost = _assign64(grid, x, A, w, power)
    J = lab.numel()
    qj = torch.ones(J, dtype=torch.int64, device=dev) if q is None else q.long()
    unit = 1.0 / J / (1.0 if q is None else 255.0)
    cnt = torch.zeros(n, dtype=torch.int64, device=dev).index_add_(0, lab, qj)
    cen = x.clone()
    rest, j = [], torch.arange(J, device=dev)
    for d in reversed(range(dim)):
        s = torch.zeros(n, dtype=torch.int64, device=dev).index_add_(0, lab, qj * (2 * (j % grid[d]) + 1))
        j = j // grid[d]
        rest.insert(0, s)
    full = cnt > 0
    for d in range(dim):
        cen[full, d] = rest[d][full].double() / cnt[full].double() * (0.5 / grid[d])
    grad = v - cnt.double() * unit
    g = (v * w).sum() + unit * (qj.double() * cost).sum()
    return {"g": float(g), "grad": grad, "maxrel": float((grad.abs() / v).max()), "counts": cnt, "centroids": cen}


def _predict64(grid, x, A, v, params):
    n = x.shape[0]
    zero = torch.zeros(n, dtype=torch.float64, device=x.device)
    d0 = n * _evaluate64(grid, x, A, v, None, zero, 2)["grad"]
    k = min(NEIGH, n - 1)
    dist = ((x[:, None, :] - x[None, :, :]) ** 2).sum(-1)
    dist.fill_diagonal_(math.inf)
    nb = dist.argsort(dim=1, stable=True)[:, :k]
    dx = x[nb] - x[:, None, :]
    Ai, Aj = A[:, None], A[nb]

    def norm2(M):
        return M[..., 0, 0] * dx[..., 0] ** 2 + 2 * M[..., 0, 1] * dx[..., 0] * dx[..., 1] + M[..., 1, 1] * dx[..., 1] ** 2

    cols = [x[:, 0], x[:, 1], A[:, 0, 0], A[:, 0, 1], A[:, 1, 1], n * v]
    cols += [math.sqrt(n) * dx[..., 0].mean(1), math.sqrt(n) * dx[..., 1].mean(1)]
    cols += [Aj[..., 0, 0].mean(1), Aj[..., 0, 1].mean(1), Aj[..., 1, 1].mean(1), n * v[nb].mean(1)]
    cols += [n * norm2(Ai).mean(1), n * norm2(Aj).mean(1)]
    cols += [math.sqrt(n) * torch.minimum(x[:, d], 1.0 - x[:, d]) for d in (0, 1)]
    cols.append(d0)
    for _ in range(3):
        cols.append(cols[-1][nb].mean(1))
    y = _layers64(params, torch.stack(cols, dim=1))
    return (y - y.mean()) / n


def _layers64(p, h):
    off = 0
    for i, o in ((FEAT, HID), (HID, HID), (HID, HID), (HID, 1)):
        h = h @ p[off:off + i * o].reshape(i, o) + p[off + i * o:off + i * o + o]
        off += i * o + o
        h = torch.relu(h) if o == HID else h[:, 0]
    return h


def exact(case, seed):
    kind = case["kind"]
    if kind in ("fit", "batch"):
        return None  # where an iteration that is stopped at 1 % ends has no exact value
    if kind == "train":
        F, t = (_dev(a) for a in _samples(case, seed))
        p = _dev(_net(seed)).requires_grad_(True)
        loss = ((_layers64(p, F) - t) ** 2).mean()
        loss.backward()
        return {"loss": float(loss.detach()), "grad": p.grad}
    x, A, v, q, w = _host(case, seed)
    x, A, v, w = _dev(x), _dev(A), _dev(v), _dev(w)
    if kind == "predict":
        return _predict64(_grid_of(case), x, A, v, _dev(_net(seed)))
    if kind == "assign":
        return _assign64(_grid_of(case), x, A, w, 2)[0]
    q = None if q is None else torch.as_tensor(q, device="cuda")
    return _evaluate64(_grid_of(case), x, A, v, q, w, case["power"])
