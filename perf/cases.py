"""Timing cases: the work a simulator built on this library has it do.

Every case goes through the public entry points of paper_1606_00556_amd.bo.
The inputs are made on the GPU from the seed alone, with the recipes of
bo_casegen (log-normal permeability, spatially correlated states, five-spot or
line-drive wells, the smooth step sequence).

Kinds
  system    one Newton system of the black-oil model as a time-stepping loop
            sees it: assembly, rebuild of the preconditioner for the new
            Jacobian in the handle's memory, FGMRES(30) to a true relative
            residual of 1e-6
  twophase  the same for the oil-water model (2x2 blocks)
  dual      the same for a dual-porosity reservoir with fixed-rate wells, the
            matrix cells eliminated exactly (condensed form)
  newton    one implicit time step: inexact Newton over such systems, on a
            grid with fixed-rate wells
  pressure  one scalar pressure system: RAS factors for new coefficients and
            90 GMRES(30) iterations
  spmv      a true residual r = b - A x on the caller's BSR matrix
  nn_fwd    the learned correction over a whole grid
  nn_train  one training step on a batch of crops: forward, loss and
            gradients, Adam
"""
import math

import numpy as np
import torch

import bo_casegen as cg
from paper_1606_00556_amd import bo as B

PREC = {"fp64": B.BO_PREC_FP64, "fp32": B.BO_PREC_FP32, "bf16": B.BO_PREC_FP32_BF16}


def listed():
    return [
        # the smallest whole call: a sector model of 2000 cells, launches and host reads count
        dict(name="system_20x20x5", kind="system", nx=20, ny=20, nz=5, sigma=1.0, day=0, precision="fp64",
             fstage="tiled", sweeps=1, fpf=0),
        # an ordinary field model with the library's FP64 preconditioner
        dict(name="system_100x100x50", kind="system", nx=100, ny=100, nz=50, sigma=1.0, day=9, precision="fp64",
             fstage="tiled", sweeps=2, fpf=0),
        # a large high-contrast model, mixed precision (FP32 cycle, BF16 factors)
        dict(name="system_200x200x50_bf16", kind="system", nx=200, ny=200, nz=50, sigma=2.0, day=3, precision="bf16",
             fstage="tiled", sweeps=2, fpf=0),
        # natural-order ILU(0) of the whole system as the second stage, on a ragged grid
        dict(name="system_99x101x31_natural", kind="system", nx=99, ny=101, nz=31, sigma=1.0, day=6, precision="fp64",
             fstage="natural", sweeps=2, fpf=0),
        # the largest model one GPU is used for: 32M dual-porosity cells
        dict(name="dual_400x400x100", kind="dual", nx=400, ny=400, nz=100, day=3),
        # one implicit time step of a ragged medium model with rate-controlled wells
        dict(name="newton_57x43x21", kind="newton", nx=57, ny=43, nz=21, sigma=1.0, dt=5.0),
        # a large oil-water model
        dict(name="twophase_200x200x50", kind="twophase", nx=200, ny=200, nz=50, sigma=2.0, day=6, sweeps=2),
        # one process's share of a 3e9-unknown pressure system
        dict(name="pressure_125x125x47", kind="pressure", nx=125, ny=125, nz=47),
        # the residual of an odd-sized model on the interchange (BSR) layout
        dict(name="spmv_197x203x51", kind="spmv", nx=197, ny=203, nz=51, sigma=1.0),
        # inference over a 2M-cell grid
        dict(name="nn_fwd_200x200x50", kind="nn_fwd", nb=1, nx=200, ny=200, nz=50),
        # the training loop's step: four crops of 32x64x64
        dict(name="nn_train_4x32x64x64", kind="nn_train", nb=4, nx=64, ny=64, nz=32, weighted=False),
        # a ragged batch with the loss weighted by the pressure matrix
        dict(name="nn_train_3x21x45x37_w", kind="nn_train", nb=3, nx=37, ny=45, nz=21, weighted=True),
    ]


def _sides(rng, lo, hi, nz_lo=4, nz_hi=60):
    """A grid of about a log-uniform number of cells between lo and hi."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    nz = max(nz_lo, min(nz_hi, int(round(math.exp(rng.uniform(math.log(nz_lo), math.log(nz_hi)))))))
    area = max(n / nz, 36.0)
    nx = max(6, int(round(math.sqrt(area) * math.exp(rng.uniform(-0.4, 0.4)))))
    ny = max(6, int(area / nx))
    while nx * ny * nz > hi:
        nx -= 1
    return nx, ny, nz


def draw(rng):
    kind = rng.choice(["system", "system", "natural", "dual", "newton", "twophase", "pressure", "spmv", "nn_fwd",
                       "nn_train"])
    if kind == "system":
        nx, ny, nz = _sides(rng, 2e3, 2e6)
        return dict(kind="system", nx=nx, ny=ny, nz=nz, sigma=rng.choice([1.0, 1.5]), day=3 * rng.randint(0, 6),
                    precision=rng.choice(["fp64", "fp64", "fp32", "bf16"]), fstage="tiled", sweeps=rng.randint(1, 2),
                    fpf=rng.randint(0, 1))
    if kind == "natural":
        nx, ny, nz = _sides(rng, 2e3, 4e5)
        return dict(kind="system", nx=nx, ny=ny, nz=nz, sigma=1.0, day=3 * rng.randint(0, 6), precision="fp64",
                    fstage="natural", sweeps=rng.randint(1, 2), fpf=rng.randint(0, 1))
    if kind == "dual":
        nx, ny, nz = _sides(rng, 5e4, 1.6e7, 8, 100)
        return dict(kind="dual", nx=max(nx, 24), ny=min(max(ny, 24), 400), nz=nz, day=3)
    if kind == "newton":
        nx, ny, nz = _sides(rng, 4e3, 1.5e5, 4, 30)
        return dict(kind="newton", nx=nx, ny=ny, nz=nz, sigma=1.0, dt=rng.choice([1.0, 3.0, 5.0]))
    if kind == "twophase":
        nx, ny, nz = _sides(rng, 2e3, 2e6)
        return dict(kind="twophase", nx=nx, ny=ny, nz=nz, sigma=rng.choice([1.0, 2.0]), day=3 * rng.randint(0, 6),
                    sweeps=rng.randint(1, 2))
    if kind == "pressure":
        nx, ny, nz = _sides(rng, 2e4, 4e6)
        return dict(kind="pressure", nx=nx, ny=ny, nz=nz)
    if kind == "spmv":
        nx, ny, nz = _sides(rng, 1e3, 4e6)
        return dict(kind="spmv", nx=nx, ny=ny, nz=nz, sigma=1.0)
    if kind == "nn_fwd":
        nx, ny, nz = _sides(rng, 5e3, 2e6)
        return dict(kind="nn_fwd", nb=1, nx=nx, ny=ny, nz=nz)
    return dict(kind="nn_train", nb=rng.randint(1, 6), nx=rng.randint(9, 64), ny=rng.randint(9, 64),
                nz=rng.randint(5, 32), weighted=rng.random() < 0.5)


# ---- inputs ---------------------------------------------------------------------
def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(1000003 * (int(seed) + 1) + salt)


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _lerp_axis(a, n, step, dim):
    f = (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / step
    i = torch.floor(f).long()
    t = f - i
    shape = [1, 1, 1]
    shape[dim] = n
    t = t.reshape(shape)
    return a.index_select(dim, i) * (1.0 - t) + a.index_select(dim, i + 1) * t


def _smooth(g, nx, ny, nz):
    """Correlated noise in [-1, 1]: uniform values every 8x8x4 cells, trilinear in between."""
    lat = 2.0 * _uniform(g, nz // 4 + 2, ny // 8 + 2, nx // 8 + 2) - 1.0
    return _lerp_axis(_lerp_axis(_lerp_axis(lat, nz, 4, 0), ny, 8, 1), nx, 8, 2).reshape(-1)


def _lognormal(g, n, mean, sigma):
    return torch.exp(math.log(mean) + sigma * torch.randn(n, generator=g, device="cuda", dtype=torch.float64))


def _base_state(g, nx, ny, nz):
    n = nx * ny * nz
    x = torch.empty(n, 3, device="cuda", dtype=torch.float64)
    for q, v in enumerate((3000.0, 0.25, 0.05)):
        x[:, q] = v * (1.0 + 0.05 * _smooth(g, nx, ny, nz))
    return x


def _state_at(base, nx, ny, nz, wells, t):
    """The smooth step sequence: pressure rises near injectors and falls near
    producers, a water front grows from the injectors."""
    if t <= 0.0:
        return base.clone()
    d = 50.0
    i = (torch.arange(nx, device="cuda", dtype=torch.float64) + 0.5)[None, :] * d
    j = (torch.arange(ny, device="cuda", dtype=torch.float64) + 0.5)[:, None] * d
    dist = {k: [torch.hypot(i - (w.i + 0.5) * d, j - (w.j + 0.5) * d) for w in wells if w.kind == k]
            for k in ("inj", "prod")}
    L = 0.2 * nx * d
    shape = sum(torch.exp(-q / L) for q in dist["inj"]) - sum(torch.exp(-q / L) for q in dist["prod"])
    front = 0.5 * (1.0 - torch.tanh((torch.stack(dist["inj"]).amin(0) - 0.3 * nx * d * math.sqrt(t / 30.0)) / (3.0 * d)))
    x = base.clone().reshape(nz, ny * nx, 3)
    x[..., 0] += 300.0 * (1.0 - math.exp(-t / 10.0)) * shape.reshape(-1)
    x[..., 1] += (0.75 - x[..., 1]) * front.reshape(-1)
    return x.reshape(-1, 3)


def _five_spot(nx, ny, nz):
    W = cg.Well
    return [W(i, j, 0, nz - 1, "inj", "bhp", 3500.0)
            for i, j in ((0, 0), (nx - 1, 0), (0, ny - 1), (nx - 1, ny - 1))] + \
           [W(nx // 2, ny // 2, 0, nz - 1, "prod", "bhp", 2500.0)]


def _rate_wells(nx, ny, nz):
    """A corner injector and a corner producer at fixed rates, and one of each at fixed pressure."""
    W = cg.Well
    return [W(0, 0, 0, nz - 1, "inj", "wrat", 800.0), W(nx - 1, ny - 1, 0, nz - 1, "prod", "lrat", 800.0),
            W(nx - 1, 0, 0, nz - 1, "inj", "bhp", 3300.0), W(nx // 2, ny // 2, 0, nz - 1, "prod", "bhp", 2700.0)]


def _case(nx, ny, nz, kx, kz, phi, wells, x_old, x_new, dt, **kw):
    return cg.Case("timing", nx, ny, nz, 50.0, 50.0, 10.0, 8000.0, kx, kx, kz, phi, x_old, x_new, dt, wells,
                   dict(cg.FLUID), **kw)


def _rock(g, c):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    n = nx * ny * nz
    kx = _lognormal(g, n, 100.0, c["sigma"])
    kz = 0.1 * kx
    if c["sigma"] >= 2.0 and nz > 8:   # thin tight layers
        for k in range(8, nz, 9):
            kx[k * nx * ny:(k + 1) * nx * ny] = 0.01
            kz[k * nx * ny:(k + 1) * nx * ny] = 0.01
    return kx, kz, 0.15 + 0.10 * _uniform(g, n)


def _single(c, seed):
    g = _gen(seed)
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    kx, kz, phi = _rock(g, c)
    wells = _five_spot(nx, ny, nz)
    base = _base_state(g, nx, ny, nz)
    t = float(c.get("day", 0))
    return _case(nx, ny, nz, kx, kz, phi, wells, _state_at(base, nx, ny, nz, wells, t).reshape(-1),
                 _state_at(base, nx, ny, nz, wells, t + 3.0 if t > 0 else 0.0).reshape(-1), 3.0 if t > 0 else 1.0)


def _dual_case(c, seed):
    g = _gen(seed)
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    n = nx * ny * nz
    lines = [int(round(f * ny)) for f in (0.125, 0.375, 0.625, 0.875)]
    cols = [int(round(f * nx)) for f in (0.1, 0.3, 0.5, 0.7, 0.9)]
    # which wells are rate controlled is part of the field's development plan, not of the seed
    wells = cg.line_drive_wells(cg.base_seed(4), nx, ny, nz, lines, cols, max(nx // 40, 1))
    kx = _lognormal(g, n, 500.0, 1.0)
    km = _lognormal(g, n, 1.0, 1.0)
    base = _base_state(g, nx, ny, nz)
    t = float(c["day"])
    xo, xn = _state_at(base, nx, ny, nz, wells, t - 3.0), _state_at(base, nx, ny, nz, wells, t)
    del base
    mn = xo.clone()
    mn[:, 0] *= 1.0 + 0.02 * (_smooth(g, nx, ny, nz) - 0.5)
    mo = mn.clone()
    mo[:, 0] -= 0.5 * (xn[:, 0] - xo[:, 0])
    ph = torch.tensor([[3200.0 if w.kind == "inj" else 2800.0, 0.0, 0.0] for w in wells if w.control != "bhp"],
                      dtype=torch.float64, device="cuda").reshape(-1, 3)
    return _case(nx, ny, nz, kx, 0.1 * kx, torch.full((n,), cg.PHI_F, dtype=torch.float64, device="cuda"), wells,
                 torch.cat([xo, mo, ph]).reshape(-1), torch.cat([xn, mn, ph]).reshape(-1), 3.0, dual=True, km=km,
                 phim=0.15 + 0.10 * _uniform(g, n), sigma=cg.kazemi_sigma())


def _pressure_system(c, seed):
    """7-point M-matrix with log-normal face coefficients, accumulation and five-spot well terms."""
    g = _gen(seed)
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    z = 1.5 * torch.randn(nz, ny, nx, generator=g, device="cuda", dtype=torch.float64)
    coef = torch.zeros(7, nz, ny, nx, dtype=torch.float64, device="cuda")
    for lo, hi, dim, s in ((0, 6, 0, 2.5), (1, 5, 1, 1.0), (2, 4, 2, 1.0)):
        m = z.shape[dim] - 1
        t = -s * torch.exp(0.5 * (z.narrow(dim, 0, m) + z.narrow(dim, 1, m)))
        coef[lo].narrow(dim, 1, m).copy_(t)
        coef[hi].narrow(dim, 0, m).copy_(t)
    acc = 1e-3 * (0.5 + _uniform(g, nz, ny, nx))
    b = acc * 3000.0 * (1.0 + 0.05 * (2.0 * _uniform(g, nz, ny, nx) - 1.0))
    coef[3] = acc - coef.sum(0)
    for w in _five_spot(nx, ny, nz):
        coef[3, :, w.j, w.i] += 10.0
        b[:, w.j, w.i] += 10.0 * w.target
    return coef.reshape(-1).contiguous(), b.reshape(-1).contiguous()


def _nn_params(seed):
    return cg.cnn_init(1606300 + int(seed) % 100000, last_scale=1.0)


def _nn_inputs(c, seed):
    """A pressure residual concentrated on a few scales beside the standardised log-permeability."""
    g = _gen(seed)
    shape = (c["nb"], c["nz"], c["ny"], c["nx"])
    r = torch.randn(shape, generator=g, device="cuda") + \
        torch.stack([_smooth(g, c["nx"], c["ny"], c["nz"]).reshape(shape[1:]) for _ in range(shape[0])]).float()
    x = torch.stack([r / r.square().mean().sqrt(), torch.randn(shape, generator=g, device="cuda")], dim=-1).contiguous()
    return x, 0.3 * r + 0.1 * torch.randn(shape, generator=g, device="cuda")


def _nn_stencil(c, seed):
    """Pressure rows scaled by their diagonal."""
    g = _gen(seed, 7)
    coef = -0.16 * torch.rand(7, c["nb"], c["nz"], c["ny"], c["nx"], generator=g, device="cuda")
    coef[3] = 1.0
    return coef.contiguous()


# ---- the calls -------------------------------------------------------------------
def prepare(case, seed):
    c, kind = case, case["kind"]
    s = dict(kind=kind)
    if kind in ("system", "dual", "twophase", "spmv"):
        cs = _dual_case(c, seed) if kind == "dual" else _single(c, seed)
        xo, xn = cs.x_old, cs.x_new
        if kind == "twophase":
            cs.fluid.update(Rs0=0.0, crs=0.0)
            xo, xn = (v.reshape(-1, 3)[:, :2].contiguous().reshape(-1) for v in (xo, xn))
            s["p"] = B.problem_from_case(cs)
            s["J"], s["b"] = B.bo_jacobian2_bsr(s["p"], xo, xo, cs.dt)
            s["pc"] = B.bo_cpr2_setup(s["J"], (cs.nx, cs.ny, cs.nz), B.bo_cpr_default_opts(sweeps=c["sweeps"]))
        else:
            s["p"] = B.problem_from_case(cs)
            s["J"], s["b"] = B.bo_jacobian_bsr(s["p"], xo, xn if kind == "spmv" else xo, cs.dt)
        if kind == "system":
            o = B.bo_cpr_default_opts(precision=PREC[c["precision"]], sweeps=c["sweeps"], fpf=c["fpf"])
            if c["fstage"] == "natural":
                o.ftype = B.BO_F_ILU_NATURAL
            s["pc"] = B.bo_cpr_setup(s["J"], (cs.nx, cs.ny, cs.nz), o)
        elif kind == "dual":
            o = B.bo_cpr_default_opts(smoother=B.BO_SMOOTH_L1, condense=1, sweeps=3, fpf=1, tile=(16, 4))
            s["pc"] = B.bo_cpr_setup(s["J"], (cs.nx, cs.ny, cs.nz, 1), o)
        s.update(xo=xo, xn=xn, dt=cs.dt, x=torch.zeros_like(s["b"]))
        if kind == "spmv":
            s["x"] = torch.randn(s["b"].numel(), generator=_gen(seed, 3), device="cuda", dtype=torch.float64)
            s["r"] = torch.empty_like(s["b"])
    elif kind == "newton":
        g = _gen(seed)
        nx, ny, nz = c["nx"], c["ny"], c["nz"]
        kx, kz, phi = _rock(g, c)
        wells = _rate_wells(nx, ny, nz)
        ph = torch.tensor([[3200.0, 0.0, 0.0], [2800.0, 0.0, 0.0]], dtype=torch.float64, device="cuda")
        x0 = torch.cat([_base_state(g, nx, ny, nz), ph]).reshape(-1)
        s["p"] = B.problem_from_case(_case(nx, ny, nz, kx, kz, phi, wells, x0, x0, c["dt"]))
        rows = nx * ny * nz + 2
        s["h"] = B.Newton(s["p"], (nx, ny, nz, 0), B.bo_cpr_default_opts(smoother=B.BO_SMOOTH_L1, npr=rows, fpf=1))
        s.update(xo=x0, x=x0.clone(), dt=c["dt"])
    elif kind == "pressure":
        s["grid"] = (c["nx"], c["ny"], c["nz"], 0)
        s["coef"], s["b"] = _pressure_system(c, seed)
        s["pc"] = B.bo_ras_setup(s["grid"], s["coef"])
        s["x"] = torch.zeros_like(s["b"])
        s["o"] = B.bo_fgmres_default_opts(flexible=0, maxit=90, rtol=1e-30)
    else:
        s["X"], s["T"] = _nn_inputs(c, seed)
        s["nn"] = B.Nn(_nn_params(seed))
        s["y"] = torch.empty_like(s["T"])
        if kind == "nn_train" and c["weighted"]:
            s["coef"] = _nn_stencil(c, seed)
    return s


def run(s):
    kind = s["kind"]
    if kind in ("system", "dual"):
        B.bo_jacobian_bsr(s["p"], s["xo"], s["xn"], s["dt"], s["J"], s["b"])
        B.bo_cpr_update(s["pc"], s["J"])
        s["x"].zero_()
        B.bo_fgmres_solve(s["pc"], s["J"], s["b"], s["x"])
        return s["J"].val, s["b"], s["x"]
    if kind == "twophase":
        B.bo_jacobian2_bsr(s["p"], s["xo"], s["xn"], s["dt"], s["J"], s["b"])
        B.bo_cpr2_update(s["pc"], s["J"])
        s["x"].zero_()
        B.bo_fgmres_solve2(s["pc"], s["J"], s["b"], s["x"])
        return s["J"].val, s["b"], s["x"]
    if kind == "newton":
        s["x"].copy_(s["xo"])
        B.bo_newton_solve(s["h"], s["xo"], s["x"], s["dt"])
        return s["x"]
    if kind == "pressure":
        B.bo_ras_update(s["pc"], s["coef"])
        s["x"].zero_()
        B.bo_scalar_solve(s["pc"], s["coef"], s["b"], s["x"], s["o"])
        return s["x"]
    if kind == "spmv":
        s["r"].copy_(s["b"])
        return B.bo_bsr_spmv(s["J"], -1.0, s["x"], 1.0, s["r"])
    s["nn"].forward(s["X"], s["y"])
    if kind == "nn_fwd":
        return s["y"]
    loss = s["nn"].backward_weighted(s["coef"], s["T"]) if "coef" in s else s["nn"].backward(s["T"])
    s["nn"].adam_step(1e-4)
    params, grads = s["nn"].get()
    return dict(y=s["y"], loss=loss, params=params, grads=grads)


# ---- the least work, and values in 64 bits ---------------------------------------
def _blocks(c):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    return nx * ny * nz + 2 * ((nx - 1) * ny * nz + nx * (ny - 1) * nz + nx * ny * (nz - 1))


def work(case):
    """Inputs read once, outputs written once; of an iterative solve one pass
    over the operator is counted, since the number of iterations is not given
    (the pressure solve's is: 90)."""
    c, kind = case, case["kind"]
    n, m = c["nx"] * c["ny"] * c["nz"], _blocks(c)
    if kind in ("system", "newton"):
        return dict(bytes=n * (32 + 48 + 24 + 24) + 2 * 72 * m, flops=40 * m)
    if kind == "dual":   # fracture stencil, and three blocks per fracture-matrix pair
        return dict(bytes=n * (48 + 96 + 48 + 48) + 2 * 72 * (m + 3 * n), flops=40 * (m + 3 * n))
    if kind == "twophase":
        return dict(bytes=n * (32 + 32 + 16 + 16) + 2 * 32 * m, flops=20 * m)
    if kind == "pressure":
        return dict(bytes=90 * 72 * n, flops=90 * 40 * n)
    if kind == "spmv":
        return dict(bytes=76 * m + n * (4 + 72), flops=18 * m)
    v = c["nb"] * n
    taps = 2 * 27 * (2 * 16 + 16 * 16 + 16 * 16 + 16)
    if kind == "nn_fwd":
        return dict(bytes=12 * v, flops=taps * v)
    return dict(bytes=(16 + (28 if c["weighted"] else 0)) * v, flops=3 * taps * v)


def _net64(params, x):
    """The network in FP64 as 27 shifted products per layer."""
    nb, nz, ny, nx, _ = x.shape
    for l, (W, b) in enumerate(params):
        p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
        y = b
        for t in range(27):
            dz, dy, dx = t // 9, (t // 3) % 3, t % 3
            y = y + torch.mm(p[:, dz:dz + nz, dy:dy + ny, dx:dx + nx].reshape(-1, W.shape[1]), W[t])
        x = y.reshape(nb, nz, ny, nx, -1)
        if l < 3:
            x = torch.relu(x)
    return x[..., 0]


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "spmv":
        # the Jacobian itself is the case's input
        s = prepare(case, seed)
        rp = s["J"].rowptr.long()
        rows = torch.repeat_interleave(torch.arange(rp.numel() - 1, device="cuda"), rp[1:] - rp[:-1])
        xv = s["x"].reshape(-1, 3)[s["J"].colind.long()]
        y = torch.zeros_like(s["b"]).reshape(-1, 3)
        y.index_add_(0, rows, (s["J"].val.reshape(-1, 3, 3) * xv[:, None, :]).sum(-1))
        return s["b"] - y.reshape(-1)
    if kind not in ("nn_fwd", "nn_train"):
        return None
    X, T = _nn_inputs(c, seed)
    train = kind == "nn_train"
    params = [(torch.from_numpy(W).double().cuda().requires_grad_(train),
               torch.from_numpy(b).double().cuda().requires_grad_(train)) for W, b in _nn_params(seed)]
    y = _net64(params, X.double())
    if not train:
        return y
    d = y - T.double()
    if c["weighted"]:
        k = _nn_stencil(c, seed).double()
        i = (slice(None),) + (slice(1, -1),) * 3
        r = k[3][i] * d[i]
        for q, (dim, sh) in enumerate(((1, -1), (2, -1), (3, -1), (0, 0), (3, 1), (2, 1), (1, 1))):
            if q != 3:
                r = r + k[q][i] * torch.roll(d, -sh, dim)[i]
        loss = r.square().mean()
    else:
        loss = d.square().mean()
    loss.backward()
    g = torch.cat([torch.cat([W.grad.reshape(-1), b.grad]) for W, b in params]).cpu().numpy()
    w = torch.cat([torch.cat([W.detach().reshape(-1), b.detach()]) for W, b in params]).cpu().numpy()
    # the first Adam step: m / (1 - 0.9) = g, v / (1 - 0.999) = g^2
    return dict(y=y.detach(), loss=float(loss), params=w - 1e-4 * g / (np.abs(g) + 1e-8), grads=g)
