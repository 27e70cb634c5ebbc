"""Performance cases of the library: the calls its users make, over the range of
sizes, types and options they make them with.

``listed()`` names the fixed cases, ``draw(rng)`` gives one more of the same
ranges; ``prepare``, ``run``, ``work`` and ``exact`` take a case (a dict of
plain values).  Kinds of cases:

  lattice     observations of one lattice in device memory -> context, solve,
              posterior (``gabp_create``, ``gabp_solve``, ``gabp_posterior``)
  multigrid   one lattice coarse to fine (``multigrid.multigrid_solve``)
  batch       many uneven lattices at once (``gabp_batch_*``)
  spacetime   the heat-equation solver (``gabp_st_*``)
  predict     the learned warm start's inference (``warm.predict``)
  train       one optimiser step of the warm-start network
  layer       one convolution, forward and backward (``gabp_conv3x3_*``)

Truth fields are plane waves evaluated at the observed cells only, so that
the largest lattices are drawn in well under a second.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

import paper_2404_12968_amd.gabp as G
import paper_2404_12968_amd.inputs as I
import paper_2404_12968_amd.multigrid as MG
import paper_2404_12968_amd.warm as W

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(W.__file__)), "weights", "warm1024.npz")
NEU, PER, DIR = I.BC_NEUMANN, I.BC_PERIODIC, I.BC_DIRICHLET


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

def _lattice(nx, ny, alpha, dtype, iters, *, bc_x=NEU, bc_y=NEU, kappa=0.2, frac=0.05, tracks=0,
             run=4, sigma=0.05, tol=1e-6, check=-10, slots=0):
    return dict(kind="lattice", nx=nx, ny=ny, alpha=alpha, dtype=dtype, iters=iters, bc_x=bc_x,
                bc_y=bc_y, kappa=kappa, frac=frac, tracks=tracks, run=run, sigma=sigma, tol=tol,
                check=check, slots=slots)


def listed():
    return [
        # the smallest whole solve: the 64 x 64 double-precision lattice to
        # 1e-10, a chain of small launches
        dict(_lattice(64, 64, 1, "f64", 2000, sigma=0.1, tol=1e-10, check=10), name="lattice64_f64"),
        # an odd-sized regional lattice, paper prior, solved for a few hundred iterations
        dict(_lattice(261, 187, 2, "f32", 600, bc_x=DIR, bc_y=DIR, kappa=0.1, frac=0.1,
                      slots=64), name="lattice261x187"),
        # double precision with the 13-point prior: the reference runs that
        # single-precision results are held against
        dict(_lattice(1030, 1000, 2, "f64", 150, kappa=0.1), name="lattice1030_f64"),
        # 2048 x 2048 along satellite tracks
        dict(_lattice(2048, 2048, 2, "f32", 300, kappa=0.05, tracks=40), name="lattice2048"),
        # the global lattice, periodic in longitude: the largest single lattice
        dict(_lattice(8192, 4096, 2, "f32", 300, bc_x=PER, kappa=0.02, tracks=60, run=7),
             name="lattice8192"),
        # the synthetic experiment's 256 x 256 grid solved coarse to fine
        dict(kind="multigrid", n=256, frac=0.1, iters=3000, name="multigrid256"),
        # many uneven instances at once
        dict(kind="batch", count=24, side_lo=64, side_hi=400, iters=400, name="batch24"),
        # a small space-time window with odd sides, every phase of the solver
        dict(kind="spacetime", nx=100, ny=75, nt=12, iters=400, dtype="f32", frac=0.03, slots=64,
             bc_x=NEU, bc_y=NEU, name="spacetime100x75x12"),
        # the full space-time workload: 64 slices of 512 x 512
        dict(kind="spacetime", nx=512, ny=512, nt=64, iters=300, dtype="f32", frac=0.02, slots=64,
             bc_x=NEU, bc_y=NEU, name="spacetime512x512x64"),
        # warm-start inference for one 1024 x 1024 problem
        dict(kind="predict", nx=1024, ny=1024, tracks=16, run=4, name="predict1024"),
        # one training step on eight 256 x 256 crops
        dict(kind="train", batch=8, ny=256, nx=256, name="train8x256"),
        # one layer on a small batch of odd size, forward and backward: the
        # smallest calls of the network path
        dict(kind="layer", batch=2, ny=61, nx=93, cin=32, cout=32, dil=9, relu=True,
             name="layer61x93"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lattice", "lattice", "lattice", "lattice", "multigrid", "batch",
                       "spacetime", "spacetime", "predict", "train", "layer", "layer"])
    if kind == "lattice":
        dtype = rng.choice(["f32", "f32", "f32", "f64"])
        most = 16e6 if dtype == "f32" else 2e6
        while True:
            nx, ny = _log(rng, 24, 8192), _log(rng, 24, 4096)
            if nx * ny <= most:
                break
        tracks = max(4, int(0.06 * nx / 4)) if nx * ny > 1e6 or rng.random() < 0.3 else 0
        return _lattice(nx, ny, rng.choice([1, 2, 2]), dtype, _log(rng, 40, 600),
                        bc_x=rng.choice([NEU, PER, DIR]), bc_y=rng.choice([NEU, PER, DIR]),
                        kappa=round(rng.uniform(0.03, 0.3), 4), frac=round(rng.uniform(0.01, 0.2), 4),
                        tracks=tracks, sigma=round(rng.uniform(0.02, 0.2), 4),
                        check=rng.choice([-10, -10, 10]), slots=rng.choice([0, 64]))
    if kind == "multigrid":
        return dict(kind=kind, n=_log(rng, 70, 512), frac=round(rng.uniform(0.08, 0.2), 4),
                    iters=_log(rng, 300, 3000))
    if kind == "batch":
        return dict(kind=kind, count=rng.randrange(3, 25), side_lo=rng.randrange(20, 100),
                    side_hi=rng.randrange(120, 400), iters=_log(rng, 40, 400))
    if kind == "spacetime":
        while True:
            nx, ny, nt = _log(rng, 16, 512), _log(rng, 16, 512), _log(rng, 2, 64)
            if nx * ny * nt <= 3e6:
                break
        return dict(kind=kind, nx=nx, ny=ny, nt=nt, iters=_log(rng, 40, 400),
                    dtype=rng.choice(["f32", "f32", "f64"]), frac=round(rng.uniform(0.01, 0.1), 4),
                    slots=rng.choice([0, 64]), bc_x=rng.choice([NEU, PER]), bc_y=rng.choice([NEU, PER]))
    if kind == "predict":
        nx, ny = _log(rng, 48, 1500), _log(rng, 48, 1024)
        return dict(kind=kind, nx=nx, ny=ny, tracks=max(2, nx // 64), run=4)
    if kind == "train":
        return dict(kind=kind, batch=rng.randrange(1, 9), ny=_log(rng, 48, 256), nx=_log(rng, 48, 256))
    return dict(kind=kind, batch=rng.randrange(1, 5), ny=_log(rng, 16, 512), nx=_log(rng, 16, 512),
                cin=rng.choice([16, 32, 32]), cout=rng.choice([16, 32, 32]),
                dil=rng.choice([1, 3, 9, 27]), relu=rng.random() < 0.8)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _waves(coords, sizes, rng, n_modes=12, max_freq=5):
    """Sum of random plane waves at integer points (one coordinate array per axis)."""
    out = np.zeros(coords[0].size)
    for _ in range(n_modes):
        arg = np.full(coords[0].size, rng.uniform(0.0, 2.0 * np.pi))
        for v, n in zip(coords, sizes):
            arg += (2.0 * np.pi * rng.integers(-max_freq, max_freq + 1) / n) * v
        out += rng.normal(0.0, np.sqrt(1.0 / n_modes)) * np.cos(arg)
    return out


def _lattice_obs(nx, ny, tracks, run, frac, sigma, seed):
    rng = np.random.default_rng(seed)
    cells = I.track_cells(nx, ny, tracks, run, rng) if tracks else I.uniform_cells(nx * ny, frac, rng)
    y = _waves((cells % nx, cells // nx), (nx, ny), rng) + sigma * rng.standard_normal(cells.size)
    return cells, y


def _st_problem(case, seed):
    nx, ny, nt = case["nx"], case["ny"], case["nt"]
    rng = np.random.default_rng(seed)
    n = nx * ny * nt
    cells = np.unique(rng.integers(0, n, size=max(1, int(case["frac"] * n))))
    t, r = np.divmod(cells, nx * ny)
    y = _waves((r % nx, r // nx, t), (nx, ny, nt), rng, max_freq=2) + 0.05 * rng.standard_normal(cells.size)
    return I.SpaceTimeProblem("st", nx, ny, nt, case["bc_x"], case["bc_y"], c=I.SPACETIME_C,
                              sigma=0.05, cells=cells, y=y, dtype=case["dtype"],
                              damping=I.SPACETIME_ETA, **I.SPACETIME_PRIOR)


def _mg_problem(case, seed):
    return I.table1(case["n"], case["frac"], instance=seed)


def _batch_problems(case, seed):
    """Instances of the uneven batch: shapes and priors of the case, data of the seed."""
    shape = np.random.default_rng(case["count"])
    probs = []
    for k in range(case["count"]):
        nx, ny = (int(v) for v in shape.integers(case["side_lo"], case["side_hi"] + 1, size=2))
        alpha, kappa = int(shape.integers(1, 3)), float(shape.uniform(0.02, 0.3))
        frac, sigma = float(shape.uniform(0.01, 0.2)), float(shape.uniform(0.02, 0.2))
        cells, y = _lattice_obs(nx, ny, 0, 0, frac, sigma, 1000 * seed + k)
        probs.append(I.Problem(f"batch[{k}]", nx, ny, NEU, NEU, alpha, kappa, 1.0,
                               I.DEFAULT_C[alpha], sigma, cells, y))
    return probs


def _predict_problem(case, seed):
    nx, ny = case["nx"], case["ny"]
    cells, y = _lattice_obs(nx, ny, case["tracks"], case["run"], 0.0, 0.05, seed)
    kappa = float(np.random.default_rng(seed).uniform(0.02, 0.3))
    return I.Problem("predict", nx, ny, NEU, NEU, 2, kappa, 1.0, 10.0, 0.05, cells, y)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _train_inputs(case, seed):
    """Network input as gabp_warm_features lays it out, and targets of the
    solver's kind: smooth means, log precisions on every edge."""
    B, H, Wd = case["batch"], case["ny"], case["nx"]
    g = _generator(seed)
    mu = torch.zeros(B, H, Wd, device="cuda")
    yy = torch.arange(H, device="cuda").view(1, H, 1) / H
    xx = torch.arange(Wd, device="cuda").view(1, 1, Wd) / Wd
    for _ in range(6):
        k = torch.randint(-3, 4, (2, B, 1, 1), generator=g, device="cuda")
        ph = 6.2832 * torch.rand(B, 1, 1, generator=g, device="cuda")
        mu += 0.4 * torch.cos(6.2832 * (k[0] * yy + k[1] * xx) + ph)
    mask = (torch.rand(B, H, Wd, generator=g, device="cuda") < 0.06).float()
    x = torch.zeros(B, H, Wd, 16, dtype=torch.bfloat16, device="cuda")
    x[..., 0] = mask.to(torch.bfloat16)
    x[..., 1] = (mask * (mu + 0.05 * torch.randn(mu.shape, generator=g, device="cuda"))).to(torch.bfloat16)
    x[..., 2] = 2.5 + torch.log(0.02 + 0.28 * torch.rand(B, 1, 1, generator=g, device="cuda")).to(torch.bfloat16)
    lam = 0.3 * torch.randn(12, B * H * Wd, generator=g, device="cuda") - 2.0
    valid = (torch.rand(12, B * H * Wd, generator=g, device="cuda") < 0.95).float()
    return x.contiguous(), mu.reshape(-1).contiguous(), lam, valid


def _train_net(seed):
    """The network in the middle of its training: trained weights, moments of
    earlier steps."""
    net = W.WarmNet.load(WEIGHTS)
    g = _generator(seed + 77)
    for m, v in zip(net.m, net.v):
        m.copy_(1e-3 * torch.randn(m.shape, generator=g, device="cuda"))
        v.copy_(1e-4 * (0.5 + torch.rand(v.shape, generator=g, device="cuda")))
    net.step = 1000
    return net


TRAIN_LR, TRAIN_LAM = 1e-3, 0.1


def _layer_inputs(case, seed):
    g = _generator(seed)
    shape = (case["batch"], case["ny"], case["nx"])
    cin, cout = case["cin"], case["cout"]
    x = torch.randn(shape + (cin,), generator=g, device="cuda").clamp_(min=0).to(torch.bfloat16)
    w = torch.zeros(32, 9 * cin, device="cuda")
    w[:cout] = math.sqrt(2.0 / (9 * cin)) * torch.randn(cout, 9 * cin, generator=g, device="cuda")
    b = torch.zeros(32, device="cuda")
    b[:cout] = 0.1 * torch.randn(cout, generator=g, device="cuda")
    dy = 1e-3 * torch.randn(shape + (cout,), generator=g, device="cuda")
    return x, w.to(torch.bfloat16), b, dy


def prepare(case, seed):
    kind = case["kind"]
    if kind == "lattice":
        cells, y = _lattice_obs(case["nx"], case["ny"], case["tracks"], case["run"], case["frac"],
                                case["sigma"], seed)
        return dict(case=case, cells=torch.from_numpy(cells).cuda(), y=torch.from_numpy(y).cuda())
    if kind == "multigrid":
        return dict(case=case, prob=_mg_problem(case, seed))
    if kind == "batch":
        return dict(case=case, probs=_batch_problems(case, seed))
    if kind == "spacetime":
        p = _st_problem(case, seed)
        return dict(case=case, prob=p, model=G.st_model(p), cells=torch.from_numpy(p.cells).cuda(),
                    y=torch.from_numpy(p.y).cuda())
    if kind == "predict":
        return dict(case=case, prob=_predict_problem(case, seed), net=W.WarmNet.load(WEIGHTS))
    if kind == "train":
        return dict(case=case, data=_train_inputs(case, seed), net=_train_net(seed))
    return dict(case=case, data=_layer_inputs(case, seed), ws=None)


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "lattice":
        ctx = G.gabp_create(G.gabp_grid(case["nx"], case["ny"], 1.0, 1.0, case["bc_x"], case["bc_y"]),
                            G.gabp_stencil(case["alpha"], case["kappa"], 1.0,
                                           I.DEFAULT_C[case["alpha"]]),
                            state["cells"], state["y"], case["sigma"], dtype=G.DTYPES[case["dtype"]])
        if case["slots"]:
            G.gabp_set_freeze_tolerance(ctx, case["slots"], 1e-6)
        st, it, rel = G.gabp_solve(ctx, case["iters"], 0.5, case["tol"], case["check"])
        mean, var = G.gabp_posterior(ctx)
        G.gabp_destroy(ctx)
        return dict(status=st, iterations=it, residual=rel, mean=mean, var=var)
    if kind == "multigrid":
        r = MG.multigrid_solve(state["prob"], max_iters=case["iters"], keep_context=True,
                               freeze_tolerance=(64, 1e-6))
        mean, var = G.gabp_posterior(r["ctx"])
        G.gabp_destroy(r["ctx"])
        return dict(status=r["status"], iterations=[v["iterations"] for v in r["levels"]],
                    residual=r["rel"], mean=mean, var=var)
    if kind == "batch":
        b = G.gabp_batch_create(state["probs"])
        st, it, rel, sts = G.gabp_batch_solve(b, case["iters"], 0.5, 1e-6, -10)
        means = [G.gabp_batch_posterior(b, k, want_var=False)[0] for k in range(b.n)]
        G.gabp_batch_destroy(b)
        return dict(status=st, iterations=it, residuals=rel, statuses=sts, means=means)
    if kind == "spacetime":
        ctx = G.gabp_st_create(state["model"], state["cells"], state["y"], state["prob"].sigma,
                               dtype=G.DTYPES[case["dtype"]])
        if case["slots"]:
            G.gabp_st_set_freeze_tolerance(ctx, case["slots"], 1e-6)
        st, it, rel = G.gabp_st_solve(ctx, case["iters"], I.SPACETIME_ETA, 1e-6, 50)
        mean, var = G.gabp_st_posterior(ctx)
        G.gabp_st_destroy(ctx)
        return dict(status=st, iterations=it, residual=rel, mean=mean, var=var)
    if kind == "predict":
        return dict(pred=W.predict(state["net"], state["prob"]))
    if kind == "train":
        net = state["net"]
        x, mu, lam, valid = state["data"]
        acts, pred = net.forward(x)
        loss, grad = G.gabp_warm_loss(pred, mu, lam, valid, W.NDIR, TRAIN_LAM)
        dws, dbs = net.backward(acts, grad)
        net.adam(dws, dbs, TRAIN_LR)
        return dict(loss=loss, pred=pred, dw=dws, db=dbs, w=[t.clone() for t in net.w],
                    b=[t.clone() for t in net.b])
    x, w, bias, dy = state["data"]
    y, _ = G.gabp_conv3x3_fwd(x, w, bias, case["cout"], case["dil"], case["relu"])
    dw, db, dx, state["ws"] = G.gabp_conv3x3_bwd(x, y, dy, w, case["cout"], case["dil"],
                                                 case["relu"], workspace=state["ws"])
    return dict(y=y, dw=dw, db=db, dx=dx)


# --------------------------------------------------------------------------
# bytes and operations of one pass
# --------------------------------------------------------------------------

_CONV = sum(9 * ci * co * 2 for ci, co in zip(W.CIN, W.COUT))   # flops per pixel, all layers


def work(case):
    """Inputs read once and outputs written once; the operations of every
    iteration (about 10 per directed edge: sums, cavity, gain, two damped
    updates) or of every convolution.  What iterations move between on-chip
    memory and HBM is the implementation's choice and is not counted."""
    kind = case["kind"]
    if kind == "lattice":
        n = case["nx"] * case["ny"]
        obs = n * (case["frac"] if not case["tracks"] else
                   min(1.0, case["tracks"] * case["run"] / case["nx"]))
        deg = 4 if case["alpha"] == 1 else 12
        return {"bytes": 16 * obs + 16 * n, "flops": 10.0 * deg * n * case["iters"]}
    if kind == "multigrid":
        n = case["n"] ** 2
        return {"bytes": 16 * case["frac"] * n + 16 * n, "flops": 10.0 * 12 * n * case["iters"] * 4 / 3}
    if kind == "batch":
        n = case["count"] * ((case["side_lo"] + case["side_hi"]) / 2) ** 2
        return {"bytes": 16 * 0.1 * n + 8 * n, "flops": 10.0 * 8 * n * case["iters"]}
    if kind == "spacetime":
        n = case["nx"] * case["ny"] * case["nt"]
        return {"bytes": 16 * case["frac"] * n + 16 * n, "flops": 10.0 * 38 * n * case["iters"]}
    if kind == "predict":
        n = case["nx"] * case["ny"]
        return {"bytes": 64 * n + 16 * case["tracks"] * case["run"] * case["ny"], "flops": float(_CONV * n)}
    if kind == "train":
        n = case["batch"] * case["ny"] * case["nx"]
        return {"bytes": n * (32 + 64 + 4 + 12 * 8), "flops": float(n * (3 * _CONV - 9 * 16 * 32 * 2))}
    n = case["batch"] * case["ny"] * case["nx"]
    return {"bytes": n * (2 * case["cin"] + 2 * case["cout"] + 4 * case["cout"] + 4 * case["cin"]),
            "flops": 3.0 * n * 9 * case["cin"] * case["cout"] * 2}


# --------------------------------------------------------------------------
# 64-bit references in plain torch
# --------------------------------------------------------------------------
# A stencil operator is a dict {offset: field}; field[i] is its entry (i, i + offset).

def _shift(f, off, per):
    """g[i] = f[i + off], zero where i + off leaves a non-periodic axis."""
    g = torch.roll(f, [-o for o in off], dims=list(range(f.dim())))
    for ax, o in enumerate(off):
        if o and not per[ax]:
            n = f.shape[ax]
            g.narrow(ax, max(0, n - o) if o > 0 else 0, min(n, abs(o))).zero_()
    return g


def _product(A, B, per):
    C = {}
    for a, fa in A.items():
        for b, fb in B.items():
            o = tuple(i + j for i, j in zip(a, b))
            v = fa * _shift(fb, a, per)
            C[o] = C[o] + v if o in C else v
    return C


def _transpose(A, per):
    return {tuple(-i for i in o): _shift(f, tuple(-i for i in o), per) for o, f in A.items()}


def _minus_laplacian(shape, bc, h, axes):
    """-Delta_h over the given axes of a grid (zero-flux, periodic or Dirichlet)."""
    per = [b == PER for b in bc]
    one = torch.ones(shape, dtype=torch.float64, device="cuda")
    zero = tuple([0] * len(shape))
    M = {zero: torch.zeros_like(one)}
    for ax in axes:
        for s in (1, -1):
            o = tuple(s if k == ax else 0 for k in range(len(shape)))
            there = _shift(one, o, per)
            M[o] = -there / h[ax] ** 2
            M[zero] = M[zero] + (there if bc[ax] == NEU else one) / h[ax] ** 2
    return M


def _lattice_precision(ny, nx, bc_y, bc_x, hy, hx, alpha, kappa, tau):
    bc = (bc_y, bc_x)
    L = _minus_laplacian((ny, nx), bc, (hy, hx), (0, 1))
    L[(0, 0)] = L[(0, 0)] + kappa ** 2
    per = [b == PER for b in bc]
    Q = L if alpha == 1 else _product(L, L, per)
    return {o: tau * f for o, f in Q.items()}, per


def _spacetime_precision(p):
    bc = (NEU, p.bc_y, p.bc_x)
    per = [False, p.bc_y == PER, p.bc_x == PER]
    shape = (p.nt, p.ny, p.nx)
    D = _minus_laplacian(shape, bc, (1.0, p.h, p.h), (1, 2))
    first = torch.zeros(shape, dtype=torch.float64, device="cuda")
    first[0] = 1.0
    M = {}
    for o, f in D.items():
        same = 1.0 if o == (0, 0, 0) else 0.0
        M[o] = first * p.a0 * (p.kappa ** 2 * same + f) + (1 - first) * (same / p.dt + 0.5 * p.nu * f)
        M[(-1, o[1], o[2])] = (1 - first) * -(same / p.dt - 0.5 * p.nu * f)
    s = p.dt * p.h ** 2 / p.sigma_u ** 2
    return {o: s * f for o, f in _product(_transpose(M, per), M, per).items()}, per


def _observed(Q, shape, cells, y, sigma):
    zero = tuple([0] * len(shape))
    cells, y = torch.from_numpy(cells).cuda(), torch.from_numpy(y).cuda()
    d = Q.pop(zero)
    diag, b = d.reshape(-1).clone(), torch.zeros_like(d).reshape(-1)
    diag.index_add_(0, cells, torch.full_like(y, 1.0 / sigma ** 2))
    b.index_add_(0, cells, y / sigma ** 2)
    return diag.reshape(shape), b.reshape(shape)


def _apply(Q, per, diag, v):
    out = diag * v
    for o, f in Q.items():
        out += f * _shift(v, o, per)
    return out


def _gabp(Q, per, diag, b, c, eta, iters, tol, every=10):
    """Damped, re-weighted flooding belief propagation; stops at the residual."""
    offs = list(Q)
    opp = [offs.index(tuple(-i for i in o)) for o in offs]
    q = torch.stack([Q[o] for o in offs]) / c
    lam, th = torch.zeros_like(q), torch.zeros_like(q)

    def incoming(m):
        return torch.stack([_shift(m[opp[k]], offs[k], per) for k in range(len(offs))])

    def belief(lin, tin):
        return diag + c * lin.sum(0), b + c * tin.sum(0)

    nb = b.norm()
    for t in range(1, iters + 1):
        lin, tin = incoming(lam), incoming(th)
        bl, bt = belief(lin, tin)
        g = -q / (bl - lin)
        lam = (1 - eta) * lam + eta * (g * q)
        th = (1 - eta) * th + eta * (g * (bt - tin))
        del lin, tin, g
        if t % every == 0 or t == iters:
            bl, bt = belief(incoming(lam), incoming(th))
            if (_apply(Q, per, diag, bt / bl) - b).norm() <= tol * nb:
                break
    return bt / bl, 1.0 / bl


def _solve_cg(Q, per, diag, b, iters=30000):
    """Conjugate gradients with a diagonal preconditioner, to 1e-13."""
    x = torch.zeros_like(b)
    r = b.clone()
    z = r / diag
    p = z.clone()
    rz = (r * z).sum()
    stop = 1e-13 * b.norm()
    for k in range(iters):
        ap = _apply(Q, per, diag, p)
        a = rz / (p * ap).sum()
        x += a * p
        r -= a * ap
        if k % 50 == 0 and r.norm() <= stop:
            break
        z = r / diag
        new = (r * z).sum()
        p = z + (new / rz) * p
        rz = new
    return x


def _conv(x, w, dil):
    """x [B,H,W,ci], w [9,ci,co] -> [B,H,W,co] (zero padding)."""
    B, H, Wd, _ = x.shape
    pad = torch.nn.functional.pad(x, (0, 0, dil, dil, dil, dil))
    out = 0
    for t in range(9):
        oy, ox = (t // 3) * dil, (t % 3) * dil
        out = out + pad[:, oy:oy + H, ox:ox + Wd] @ w[t]
    return out


def _taps(w, cout):
    """[32, 9*cin] rows of the library's layout -> float64 [9, cin, cout]."""
    return w[:cout].double().reshape(cout, 9, -1).permute(1, 2, 0).contiguous()


def _net_forward(ws, bs, x):
    for l in range(len(W.DILATIONS)):
        x = _conv(x, ws[l], W.DILATIONS[l]) + bs[l][:W.COUT[l]]
        if W.RELU[l]:
            x = torch.relu(x)
    return x


def _rows(dw, cin):
    """Gradient [9, cin, cout] -> the library's [32, 9*cin]."""
    out = torch.zeros(32, 9 * cin, dtype=torch.float64, device="cuda")
    out[:dw.shape[2]] = dw.permute(2, 0, 1).reshape(dw.shape[2], -1)
    return out


def _exact_train(case, seed):
    net = _train_net(seed)
    x, mu, lam, valid = _train_inputs(case, seed)
    L = len(W.DILATIONS)
    ws = [_taps(net.wb[l], W.COUT[l]).requires_grad_() for l in range(L)]
    bs = [net.b[l].double().requires_grad_() for l in range(L)]
    pred = _net_forward(ws, bs, x.double())
    n = mu.numel()
    out = pred.reshape(n, 16)
    loss = ((out[:, 0] - mu.double()) ** 2).sum() / n
    loss = loss + TRAIN_LAM / (12 * n) * (((out[:, 1:13].T - lam.double()) ** 2) * (valid > 0)).sum()
    loss.backward()
    dw = [_rows(ws[l].grad, W.CIN[l]) for l in range(L)]
    db = [bs[l].grad for l in range(L)]
    new = []
    for k, (w, g) in enumerate(zip(net.w + net.b, dw + db)):
        m = 0.9 * net.m[k].double() + 0.1 * g
        v = 0.999 * net.v[k].double() + 0.001 * g * g
        t = net.step + 1
        new.append(w.double() - TRAIN_LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8))
    return dict(loss=loss.detach(), pred=pred.detach(), dw=dw, db=db, w=new[:L], b=new[L:])


def exact(case, seed):
    kind = case["kind"]
    if kind == "lattice":
        deg = 4 if case["alpha"] == 1 else 12
        if case["nx"] * case["ny"] * deg * case["iters"] > 1.5e11:
            return None
        cells, y = _lattice_obs(case["nx"], case["ny"], case["tracks"], case["run"], case["frac"],
                                case["sigma"], seed)
        Q, per = _lattice_precision(case["ny"], case["nx"], case["bc_y"], case["bc_x"], 1.0, 1.0,
                                    case["alpha"], case["kappa"], 1.0)
        diag, b = _observed(Q, (case["ny"], case["nx"]), cells, y, case["sigma"])
        mean, var = _gabp(Q, per, diag, b, I.DEFAULT_C[case["alpha"]], 0.5, case["iters"], case["tol"])
        return dict(status=None, iterations=None, residual=None, mean=mean, var=var)
    if kind == "multigrid":
        p = _mg_problem(case, seed)
        Q, per = _lattice_precision(p.ny, p.nx, p.bc_y, p.bc_x, p.hy, p.hx, 2, p.kappa, p.tau)
        diag, b = _observed(Q, (p.ny, p.nx), p.cells, p.y, p.sigma)
        levels = MG.max_levels(p)
        return dict(status=None, iterations=[None] * levels, residual=None,
                    mean=_solve_cg(Q, per, diag, b), var=None)
    if kind == "batch":
        means = []
        for p in _batch_problems(case, seed):
            Q, per = _lattice_precision(p.ny, p.nx, p.bc_y, p.bc_x, 1.0, 1.0, p.alpha, p.kappa, p.tau)
            diag, b = _observed(Q, (p.ny, p.nx), p.cells, p.y, p.sigma)
            means.append(_gabp(Q, per, diag, b, p.c, p.damping, case["iters"], 1e-6)[0])
        return dict(status=None, iterations=None, residuals=None, statuses=None, means=means)
    if kind == "spacetime":
        n = case["nx"] * case["ny"] * case["nt"]
        if n * 38 * case["iters"] > 1e11:
            return None
        p = _st_problem(case, seed)
        Q, per = _spacetime_precision(p)
        diag, b = _observed(Q, (p.nt, p.ny, p.nx), p.cells, p.y, p.sigma)
        mean, var = _gabp(Q, per, diag, b, p.c, p.damping, case["iters"], 1e-6, every=50)
        return dict(status=None, iterations=None, residual=None, mean=mean, var=var)
    if kind == "predict":
        p = _predict_problem(case, seed)
        x = torch.zeros(p.ny * p.nx, 16, dtype=torch.float64, device="cuda")
        cells = torch.from_numpy(p.cells).cuda()
        x[cells, 0] = 1.0
        x[cells, 1] = torch.from_numpy(p.y).cuda()
        x[:, 2] = math.log(p.kappa) + 2.5
        net = W.WarmNet.load(WEIGHTS)
        ws = [_taps(net.wb[l], W.COUT[l]) for l in range(len(W.DILATIONS))]
        out = _net_forward(ws, [b.double() for b in net.b], x.reshape(1, p.ny, p.nx, 16))
        return dict(pred=out[0])
    if kind == "train":
        return _exact_train(case, seed)
    x, w, bias, dy = _layer_inputs(case, seed)
    wt = _taps(w, case["cout"]).requires_grad_()
    xd = x.double().requires_grad_()
    bd = bias.double().requires_grad_()
    y = _conv(xd, wt, case["dil"]) + bd[:case["cout"]]
    if case["relu"]:
        y = torch.relu(y)
    y.backward(dy.double())
    return dict(y=y.detach(), dw=_rows(wt.grad, case["cin"]), db=bd.grad, dx=xd.grad)
