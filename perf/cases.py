"""The work that programs have this library do, as cases that can be timed.

A case is a dict of plain values: the form of the call (``form``), the medium
(``medium``, ``nx``, ``ny``, ``quad``) and the solver options. ``listed()``
gives the standing ones, ``draw()`` more of the same ranges, ``prepare()``
makes what a program holds before the call (problem tensors on the GPU; the
plan where a program keeps one), ``run()`` is one pass through the public
entry points, ``work()`` the bytes and operations a pass cannot do without,
and ``exact()`` the same outputs from a plain torch implementation in 64 bits
where the result does not depend on where an inner iteration stops.

Forms:
  plan    a kept plan restarted, ``iters`` outer iterations, fields read
  solve   gsis_solve: set-up, iterations to Err < 1e-6, fields
  batch   a kept batch of uneven problems restarted, ``iters`` iterations
  design  one step of an inverse-design loop: forward solve and gradient
          through torch autograd
  adjoint gradients of a kept, converged plan
  td      a kept time-dependent plan restarted, ``steps`` time steps
"""
import math
import random

import numpy as np
import torch

from paper_2507_03975_amd import gsis, inputs
from paper_2507_03975_amd.autograd import gsis_fixed_point

DEV = "cuda:0"
FOUR_PI = 4.0 * math.pi

# Ordinate sets: S4; Gauss-Legendre polar x Chebyshev azimuthal ("2x16" ...);
# the full Gauss-Legendre product of the 2D hot-wall experiment ("full36x48").
QUADS = {"s4": 12, "2x16": 32, "2x32": 64, "4x32": 128, "full18x24": 432, "full36x48": 1728}

PLAN = dict(form="plan", method=1, precision=0, limiter=1, beta=0.0, hot_face=0,
            synth_rtol=0.1, synth_max_iter=50)


def listed():
    return [
        # the smallest call: a one-shot solve of the S4 box (latency, set-up, launches)
        dict(name="solve_s4_32", form="solve", medium="uniform", nx=32, ny=32, quad="s4",
             limiter=1, beta=0.0, noalloc=False, work_iters=10),
        # the 2D hot-wall experiment, source iteration on its small grid: thousands of cheap
        # iterations in use, many ordinates
        dict(PLAN, name="wall_si_40x40x1728", medium="wall", nx=40, ny=40, quad="full36x48",
             method=0, limiter=0, iters=64),
        # the same experiment by GSIS on its larger grid, synthetic solves to 1e-8
        dict(PLAN, name="wall_gsis_100x100x1728", medium="wall", nx=100, ny=100,
             quad="full36x48", limiter=0, synth_rtol=1e-8, synth_max_iter=200, iters=8),
        # the benchmark workload: iterations on a kept plan, limiter on
        dict(PLAN, name="square_256x256x128", medium="square", nx=256, ny=256, quad="4x32",
             iters=10),
        # the same problem from inputs to converged fields in one call
        dict(name="solve_256x256x128", form="solve", medium="square", nx=256, ny=256,
             quad="4x32", limiter=1, beta=0.0, noalloc=False, work_iters=28),
        # a large medium of strong opacity jumps, intensities far beyond the caches
        dict(PLAN, name="blocks_1024x1024x128", medium="blocks", nx=1024, ny=1024, quad="4x32",
             limiter=0, beta=10.0, iters=4),
        # the FP32-mixed form
        dict(PLAN, name="blocks_fp32_512x512x128", medium="blocks", nx=512, ny=512, quad="4x32",
             precision=1, limiter=0, beta=10.0, iters=8),
        # an odd-sized grid with inflow on every wall and transport-face HoT
        dict(PLAN, name="random_faces_203x331x64", medium="random", nx=203, ny=331, quad="2x32",
             hot_face=1, iters=8),
        # a batch of uneven problems advanced together
        dict(name="batch_16_uneven", form="batch", count=16, lo=64, hi=256, shapes=4, iters=10),
        # inverse design: forward and gradient per step, new coefficients each time
        dict(name="design_256x256x128", form="design", medium="square", nx=256, ny=256,
             quad="4x32", work_iters=80),
        # backward pass of a kept plan at the detector problem's size
        dict(name="adjoint_512x512x128", form="adjoint", medium="square", nx=512, ny=512,
             quad="4x32", work_iters=54),
        # time steps with the material energy equation
        dict(name="td_128x128x128", form="td", medium="square", nx=128, ny=128, quad="4x32",
             method=1, limiter=1, cdt=0.01, steps=2, work_iters=18),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes log-uniform (odd ones among them), options as in use."""
    form = rng.choice(["plan", "plan", "plan", "plan", "solve", "solve", "batch", "design",
                       "adjoint", "td"])
    if form == "batch":
        return dict(form="batch", count=rng.randint(4, 16), lo=rng.choice([32, 48, 64]),
                    hi=rng.choice([128, 200, 256]), shapes=rng.randrange(1 << 20),
                    iters=rng.randint(4, 10))
    quad = rng.choice(["s4", "2x16", "2x32", "4x32", "4x32", "full18x24", "full36x48"])
    top = {"plan": 1 << 25, "solve": 1 << 23, "design": 1 << 22, "adjoint": 1 << 24,
           "td": 1 << 21}[form]
    side = min(1024, int(math.sqrt(top / QUADS[quad])))
    nx, ny = _log_int(rng, 24, side), _log_int(rng, 24, side)
    if form == "plan":
        medium = rng.choice(["wall", "square", "blocks", "random", "uniform"])
        c = dict(PLAN, medium=medium, nx=nx, ny=ny, quad=quad, method=rng.choice([0, 1, 1, 1]),
                 precision=rng.choice([0, 0, 1]), limiter=rng.choice([0, 1]),
                 iters=rng.randint(3, 10))
        if medium == "blocks":
            c.update(beta=10.0, limiter=0)
        elif c["method"] == 1 and medium in ("random", "uniform"):
            c["hot_face"] = rng.choice([0, 1])
        if c["method"] == 1 and rng.random() < 0.3:
            c.update(synth_rtol=1e-8, synth_max_iter=200)
        return c
    if form == "solve":
        medium = rng.choice(["square", "blocks", "uniform"])
        return dict(form="solve", medium=medium, nx=nx, ny=ny, quad=quad,
                    limiter=0 if medium == "blocks" else 1,
                    beta=10.0 if medium == "blocks" else 0.0,
                    noalloc=bool(nx * ny * (QUADS[quad] * 16 + 4000) < (150 << 20)
                                 and rng.random() < 0.3), work_iters=25)
    if form == "td":
        return dict(form="td", medium="square", nx=nx, ny=ny, quad=quad, method=1, limiter=1,
                    cdt=rng.choice([0.01, 0.1]), steps=rng.randint(1, 3), work_iters=16)
    return dict(form=form, medium="square", nx=nx, ny=ny, quad=quad,
                work_iters=80 if form == "design" else 54)


# ------------------------------------------------------------------- inputs
def _quad(name):
    if name == "s4":
        return inputs.quad_s4()
    a, b = (int(v) for v in name.replace("full", "").split("x"))
    return inputs.quad_gl_product_full(a, b) if name.startswith("full") else \
        inputs.quad_product(a, b)


def _problem(medium, nx, ny, quad, seed):
    """Problem dict with CUDA tensors on the unit square, random from the seed.

    wall     pure scatterer, sigma_t in [8, 20], hot bottom wall
    square   thick scattering square (optical thickness 4 per cell) in a thin
             absorber, 20 % noise per cell
    blocks   7 x 7 blocks, sigma_a logU[1e-2, 1e2], sigma_s logU[1e-1, 1e4]
    random   per-cell sigma_t logU[0.1, 10], c U[0.3, 0.95], inflow everywhere
    uniform  sigma_t = 1, c = 0.9, 20 % noise
    """
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 2654435761 % (1 << 31) + 17)
    f64 = dict(dtype=torch.float64, device=DEV)
    rand = lambda *s: torch.rand(*s, generator=g, **f64)  # noqa: E731
    mu, eta, w = (torch.from_numpy(np.ascontiguousarray(v)).to(DEV) for v in _quad(quad))
    K, N = len(mu), nx * ny
    p = dict(nx=nx, ny=ny, dx=1.0 / nx, dy=1.0 / ny, mu=mu, eta=eta, w=w, bnd_in=None)
    jj, ii = torch.meshgrid(torch.arange(ny, device=DEV), torch.arange(nx, device=DEV),
                            indexing="ij")
    if medium == "wall":
        st = 8.0 + 12.0 * float(rand(1))
        p["sigma_s"] = torch.full((N,), st, **f64)
        p["sigma_a"] = torch.zeros(N, **f64)
        p["q"] = torch.zeros(N, **f64)
        b = torch.full((2 * (nx + ny), K), 1e-6 / FOUR_PI, **f64)
        b[2 * ny:2 * ny + nx] = 1.0 / FOUR_PI
        p["bnd_in"] = b
        return p
    if medium == "square":
        inside = ((ii >= nx // 4) & (ii < 3 * nx // 4) & (jj >= ny // 4)
                  & (jj < 3 * ny // 4)).reshape(-1)
        st = torch.where(inside, 4.0 * min(nx, ny), 1.0).to(torch.float64)
        cc = torch.where(inside, 0.9999, 0.5).to(torch.float64)
        p["q"] = inside.to(torch.float64)
    elif medium == "blocks":
        sa = torch.exp(math.log(1e-2) + rand(49) * math.log(1e4))
        ss = torch.exp(math.log(1e-1) + rand(49) * math.log(1e5))
        at = ((jj * 7 // ny) * 7 + ii * 7 // nx).reshape(-1)
        p["sigma_a"], p["sigma_s"] = sa[at].contiguous(), ss[at].contiguous()
        p["q"] = torch.ones(N, **f64)
        return p
    elif medium == "random":
        st = torch.exp(math.log(0.1) + rand(N) * math.log(100.0))
        cc = 0.3 + 0.65 * rand(N)
        p["q"] = rand(N)
        p["bnd_in"] = 0.2 * rand(2 * (nx + ny), K)
        p["sigma_s"], p["sigma_a"] = cc * st, st - cc * st
        return p
    else:
        st, cc = torch.ones(N, **f64), torch.full((N,), 0.9, **f64)
        p["q"] = torch.ones(N, **f64)
    p["sigma_s"] = cc * st * (0.8 + 0.4 * rand(N))
    p["sigma_a"] = (st - cc * st) * (0.8 + 0.4 * rand(N))
    return p


def _batch_shapes(case):
    """(nx, ny, quad) of each problem of a batch: a few sizes of the range, uneven."""
    rng = random.Random(case["shapes"])
    sizes = sorted({case["lo"], case["hi"], _log_int(rng, case["lo"], case["hi"]),
                    _log_int(rng, case["lo"], case["hi"]) | 1})
    return [(rng.choice(sizes), rng.choice(sizes), rng.choice(["2x16", "2x32", "4x32"]))
            for _ in range(case["count"])]


_CTX = []


def _ctx():
    if not _CTX:
        _CTX.append(gsis.Context(0))
    return _CTX[0]


def _plan_options(case):
    return dict(method=case["method"], precision=case["precision"], limiter=case["limiter"],
                beta=case["beta"], hot_face=case["hot_face"], tol=1e-6, max_iter=1000,
                synth_rtol=case["synth_rtol"], synth_max_iter=case["synth_max_iter"])


def _detector(nx, ny, p):
    """V sigma_a on a window right of the square: dJ/dphi of the detector reading."""
    win = torch.zeros(ny, nx, dtype=torch.float64, device=DEV)
    win[(15 * ny) // 32:max((17 * ny) // 32, (15 * ny) // 32 + 1),
        (27 * nx) // 32:max((29 * nx) // 32, (27 * nx) // 32 + 1)] = p["dx"] * p["dy"]
    return win.reshape(-1)


def prepare(case, seed):
    form = case["form"]
    s = dict(case=case)
    if form == "batch":
        probs = [_problem("blocks", nx, ny, quad, seed * 100 + i)
                 for i, (nx, ny, quad) in enumerate(_batch_shapes(case))]
        s["batch"] = gsis.Batch(_ctx(), probs, tol=1e-6, max_iter=1000, limiter=0, beta=20.0)
        return s
    p = s["problem"] = _problem(case["medium"], case["nx"], case["ny"], case["quad"], seed)
    if form == "plan":
        s["plan"] = gsis.Plan(_ctx(), p, **_plan_options(case))
    elif form == "td":
        s["plan"] = gsis.TDPlan(_ctx(), p, 0.1, c=1.0, a=1.0, dt=case["cdt"], cv=1.0, sub_iter=3,
                                method=case["method"], limiter=case["limiter"], tol=1e-6,
                                max_iter=200)
    elif form == "design":
        s["window"] = _detector(case["nx"], case["ny"], p)
        s["static"] = dict({k: p[k] for k in ("nx", "ny", "dx", "dy", "mu", "eta", "w")},
                           options=dict(tol=1e-6, max_iter=400, limiter=0))
        s["param"] = [p[k].clone().requires_grad_(True) for k in ("sigma_a", "sigma_s", "q")]
    elif form == "adjoint":
        s["g"] = _detector(case["nx"], case["ny"], p) * p["sigma_a"]
        s["plan"] = gsis.Plan(_ctx(), p, limiter=0, tol=1e-6, max_iter=400)
        n, conv = 0, 0
        while conv == 0 and n < 400:
            s["plan"].iterate(16)
            n, conv, _ = s["plan"].status()
    return s


# --------------------------------------------------------------------- pass
def run(s):
    case = s["case"]
    form = case["form"]
    if form == "plan":
        plan = s["plan"]
        plan.reset()
        plan.iterate(case["iters"])
        return plan.read()
    if form == "solve":
        r = gsis.gsis_solve(_ctx(), s["problem"], noalloc=case["noalloc"], tol=1e-6,
                            max_iter=200, limiter=case["limiter"], beta=case["beta"])
        # (the histories' length is the iteration count, which the medium decides)
        return {k: r[k] for k in ("phi", "Fx", "Fy", "n_iter", "final_err")}
    if form == "batch":
        b = s["batch"]
        b.reset()
        b.iterate(case["iters"])
        out = []
        for i in range(b.n):
            r = b.read(i)
            out.append([r["phi"], r["Fx"], r["Fy"]])
        return out
    if form == "td":
        plan = s["plan"]
        plan.reset()
        status, its, errs = plan.advance(case["steps"])
        return dict(plan.read_td(), inner=its, err=errs)
    if form == "design":
        sa, ss, q = s["param"]
        phi, fx, fy = gsis_fixed_point(sa, ss, q, s["static"])
        reading = (s["window"] * sa * phi).sum()
        ga, gs, gq = torch.autograd.grad(reading, (sa, ss, q))
        return dict(phi=phi.detach(), Fx=fx.detach(), Fy=fy.detach(), reading=reading.detach(),
                    grad_sigma_a=ga, grad_sigma_s=gs, grad_q=gq)
    ga, gs, gq, info = s["plan"].adjoint(s["g"], tol=1e-6, max_iter=400)
    return dict(grad_sigma_a=ga, grad_sigma_s=gs, grad_q=gq, n_iter=info["n_iter"])


def work(case):
    """One read and one write of the intensities per outer iteration (8 B each,
    4 B in the FP32-mixed form) and about 60 operations per cell-ordinate;
    iteration counts that depend on the data are the usual ones."""
    if case["form"] == "batch":
        nk = sum(nx * ny * QUADS[q] for nx, ny, q in _batch_shapes(case))
        cells = sum(nx * ny for nx, ny, _ in _batch_shapes(case))
    else:
        nk = case["nx"] * case["ny"] * QUADS[case["quad"]]
        cells = case["nx"] * case["ny"]
    its = case.get("iters") or case["work_iters"]
    size = 4 if case.get("precision") == 1 else 8
    return {"bytes": its * (2.0 * size * nk) + 8.0 * 8 * cells, "flops": its * 60.0 * nk}


# -------------------------------------------------- the same in plain torch
def _shift(a, dim, by):
    """Neighbour values along dim (by = +1: the next cell's), the wall cells their own."""
    n = a.shape[dim]
    at = (torch.arange(n, device=a.device) + by).clamp(0, n - 1)
    return a.index_select(dim, at)


def _coefficients(st, nx, ny, dx, dy):
    """Adaptive least-squares coefficients cE, cW, cN, cS (Eqs. shifted_j, LSF_mdf)."""
    def one_dir(dim, h):
        dp = 0.5 * h + _shift(st, dim, 1) / st * (0.5 * h)
        dm = 0.5 * h + _shift(st, dim, -1) / st * (0.5 * h)
        dp.narrow(dim, dp.shape[dim] - 1, 1).zero_()
        dm.narrow(dim, 0, 1).zero_()
        m = dp * dp + dm * dm
        one = torch.where(m > 0, m, torch.ones_like(m))
        return dp / one, dm / one
    cE, cW = one_dir(1, dx)
    cN, cS = one_dir(0, dy)
    return cE, cW, cN, cS


def _out_faces(u, co, hx, hy, limiter):
    """Values on the east and north faces of every cell, flow towards +x, +y."""
    ue, uw, un, us = (_shift(u, -1, 1), _shift(u, -1, -1), _shift(u, -2, 1), _shift(u, -2, -1))
    cE, cW, cN, cS = co
    gx = (cE * (ue - u) - cW * (uw - u)) * hx
    gy = (cN * (un - u) - cS * (us - u)) * hy
    if limiter:
        hi = torch.maximum(torch.maximum(torch.maximum(u, ue), torch.maximum(uw, un)), us)
        lo = torch.minimum(torch.minimum(torch.minimum(u, ue), torch.minimum(uw, un)), us)
        m, M = torch.minimum(hi - u, u - lo), torch.maximum(gx.abs(), gy.abs())
        psi = torch.where(M > m, m / torch.where(M > 0, M, torch.ones_like(M)),
                          torch.ones_like(M))
        gx, gy = psi * gx, psi * gy
    return u + gx, u + gy


def exact(case, seed):
    """phi, F of a plan's iterate: source iteration, and GSIS with tight
    synthetic solves on grids whose synthetic matrix can be factored densely."""
    if case["form"] != "plan" or case["precision"] or case["beta"] or case["hot_face"]:
        return None
    nx, ny = case["nx"], case["ny"]
    N, K, gs = nx * ny, QUADS[case["quad"]], case["method"] == 1
    if gs and (case["synth_rtol"] > 1e-6 or N > 12000):
        return None
    if N * K > (1 << 25) or 4 * (nx + ny) * case["iters"] > 40000:
        return None
    p = _problem(case["medium"], nx, ny, case["quad"], seed)
    dx, dy = p["dx"], p["dy"]
    sa, ss, q = (p[k].reshape(ny, nx) for k in ("sigma_a", "sigma_s", "q"))
    st = sa + ss
    mu, eta, w, bnd = p["mu"], p["eta"], p["w"], p["bnd_in"]
    co = _coefficients(st, nx, ny, dx, dy)
    quads = []          # per quadrant: ordinates, flips, flipped coefficients, inflow
    for fx in (False, True):
        for fy in (False, True):
            k = torch.nonzero(((mu < 0) == fx) & ((eta < 0) == fy)).reshape(-1)
            dims = ([-1] if fx else []) + ([-2] if fy else [])
            cE, cW, cN, cS = ((co[1], co[0]) if fx else (co[0], co[1])) + \
                ((co[3], co[2]) if fy else (co[2], co[3]))
            inW = torch.zeros(len(k), ny, dtype=torch.float64, device=DEV)
            inS = torch.zeros(len(k), nx, dtype=torch.float64, device=DEV)
            if bnd is not None:
                bw = bnd[ny:2 * ny] if fx else bnd[:ny]
                bs = bnd[2 * ny + nx:] if fy else bnd[2 * ny:2 * ny + nx]
                inW, inS = bw.index_select(1, k).T, bs.index_select(1, k).T
                inW = inW.flip(-1) if fy else inW
                inS = inS.flip(-1) if fx else inS
            quads.append((k, dims, [c.flip(dims) for c in (cE, cW, cN, cS)], inW, inS))
    diag = []
    for d in range(nx + ny - 1):
        y = torch.arange(max(0, d - nx + 1), min(ny, d + 1), device=DEV)
        diag.append((y, d - y))
    if gs:
        chol, kap, ax, ay = _synthetic(sa, st, nx, ny, dx, dy)
    cur = torch.zeros(K, ny, nx, dtype=torch.float64, device=DEV)
    phi = torch.zeros(ny, nx, dtype=torch.float64, device=DEV)
    corr = torch.zeros_like(phi)
    for _ in range(case["iters"]):
        cur += corr / FOUR_PI
        src = (ss * phi + q) / FOUR_PI
        wall = torch.zeros(4, max(nx, ny), dtype=torch.float64, device=DEV)   # W, E, S, N
        for k, dims, cf, inW, inS in quads:
            u = cur[k].flip(dims)
            ox, oy = (mu[k].abs() / dx)[:, None, None], (eta[k].abs() / dy)[:, None, None]
            sf, tf = src.flip(dims), st.flip(dims)
            Fe, Fn = _out_faces(u, cf, 0.5 * dx, 0.5 * dy, case["limiter"])
            r = sf - tf * u
            r -= ox * (Fe - torch.cat([inW[:, :, None], Fe[:, :, :-1]], 2))
            r -= oy * (Fn - torch.cat([inS[:, None, :], Fn[:, :-1, :]], 1))
            dI = torch.zeros(len(k), ny + 1, nx + 1, dtype=torch.float64, device=DEV)
            dg = tf + ox + oy
            for y, x in diag:
                dI[:, y + 1, x + 1] = (r[:, y, x] + ox[:, 0] * dI[:, y + 1, x]
                                       + oy[:, 0] * dI[:, y, x + 1]) / dg[:, y, x]
            v = u + dI[:, 1:, 1:]
            cur[k] = v.flip(dims)
            if gs:       # w Omega . n_out of the reconstructed outgoing and the given incoming values
                Ge, Gn = _out_faces(v, cf, 0.5 * dx, 0.5 * dy, case["limiter"])
                fx, fy = -1 in dims, -2 in dims
                wm, we = (w * mu.abs())[k] @ torch.stack([Ge[:, :, -1], inW], 1).reshape(len(k), -1), \
                    (w * eta.abs())[k] @ torch.stack([Gn[:, -1, :], inS], 1).reshape(len(k), -1)
                (oE, iW), (oN, iS) = wm.reshape(2, ny), we.reshape(2, nx)
                oE, iW = (oE.flip(0), iW.flip(0)) if fy else (oE, iW)
                oN, iS = (oN.flip(0), iS.flip(0)) if fx else (oN, iS)
                wall[0 if fx else 1, :ny] += oE
                wall[1 if fx else 0, :ny] -= iW
                wall[2 if fy else 3, :nx] += oN
                wall[3 if fy else 2, :nx] -= iS
        half, Fx, Fy = (torch.tensordot(v, cur, 1) for v in (w, w * mu, w * eta))
        if not gs:
            phi = half
            continue
        gx = co[0] * (_shift(half, 1, 1) - half) - co[1] * (_shift(half, 1, -1) - half)
        gy = co[2] * (_shift(half, 0, 1) - half) - co[3] * (_shift(half, 0, -1) - half)
        hx, hy = Fx + gx / (3.0 * st), Fy + gy / (3.0 * st)
        b = dx * dy * q
        fe, fn = 0.5 * dy * (hx[:, 1:] + hx[:, :-1]), 0.5 * dx * (hy[1:] + hy[:-1])
        b[:, :-1] -= fe
        b[:, 1:] += fe
        b[:-1] -= fn
        b[1:] += fn
        b[:, 0] -= dy * (wall[0, :ny] - kap[0] * half[:, 0])
        b[:, -1] -= dy * (wall[1, :ny] - kap[1] * half[:, -1])
        b[0] -= dx * (wall[2, :nx] - kap[2] * half[0])
        b[-1] -= dx * (wall[3, :nx] - kap[3] * half[-1])
        phi = torch.cholesky_solve(b.reshape(-1, 1), chol).reshape(ny, nx)
        corr = phi - half
    if gs:
        Fx, Fy = Fx + corr / FOUR_PI * (w * mu).sum(), Fy + corr / FOUR_PI * (w * eta).sum()
    return dict(phi=phi.reshape(-1), Fx=Fx.reshape(-1), Fy=Fy.reshape(-1))


def _synthetic(sa, st, nx, ny, dx, dy):
    """Cholesky factor of the dense synthetic matrix, wall coefficients, couplings."""
    ax = dy * 2.0 / (3.0 * (st[:, :-1] + st[:, 1:]) * dx)
    ay = dx * 2.0 / (3.0 * (st[:-1] + st[1:]) * dy)
    kap = [2.0 / (3.0 * s * h) + 0.25 for s, h in
           ((st[:, 0], dx), (st[:, -1], dx), (st[0], dy), (st[-1], dy))]
    d = dx * dy * sa
    d[:, :-1] += ax
    d[:, 1:] += ax
    d[:-1] += ay
    d[1:] += ay
    d[:, 0] += dy * kap[0]
    d[:, -1] += dy * kap[1]
    d[0] += dx * kap[2]
    d[-1] += dx * kap[3]
    A = torch.diag(d.reshape(-1))
    c = torch.arange(nx * ny, device=DEV).reshape(ny, nx)
    for a, i, j in ((ax, c[:, :-1], c[:, 1:]), (ay, c[:-1], c[1:])):
        A[i.reshape(-1), j.reshape(-1)] = -a.reshape(-1)
        A[j.reshape(-1), i.reshape(-1)] = -a.reshape(-1)
    return torch.linalg.cholesky(A), kap, ax, ay
