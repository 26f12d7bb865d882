"""GPU: the one-workgroup multigrid cycle and the synthetic solve that runs
wholly in it (grids of at most 4096 cells), against the oracle at the sizes
where their paths change: a single cell, a dense solve alone, rows and columns,
odd widths (pairs of cells across a row's end, a last cell on its own), the
largest of each number of pairs per thread, and the first that needs a tile
level."""
import sys

import numpy as np
import pytest

import oracle
from paper_2507_03975_amd import gsis, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gsis.Context(0)


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _np(a):
    return a.cpu().numpy() if hasattr(a, "cpu") else np.asarray(a)


def _rel(a, b):
    return np.abs(_np(a) - b).max() / max(np.abs(b).max(), 1e-300)


SIZES = [(1, 1), (2, 1), (8, 8), (9, 8), (1, 300), (300, 1), (32, 32), (33, 31), (2, 511), (45, 45),
         (64, 64), (63, 65), (65, 63), (1365, 3), (2, 2047), (65, 64), (91, 46), (128, 128),
         (127, 129), (50, 50), (47, 53), (64, 48), (100, 100), (101, 97)]


@pytest.mark.parametrize("shape", SIZES)
def test_gsis_against_oracle(ctx, shape):
    """phi and F of the third iterate to 1e-10, the FP64 bound of iterates
    with a synthetic solve (converged to its rounding on both sides)."""
    p = inputs.random_problem(shape[0], shape[1], seed=5, sigma_range=(0.1, 5.0))
    _say("coarse cycle %s" % (shape,))
    g = gsis.gsis_solve(ctx, p, tol=0.0, max_iter=3, synth_rtol=1e-15, synth_max_iter=200)
    o = oracle.solve(p, tol=0.0, max_iter=3)
    for f in ("phi", "Fx", "Fy"):
        s = max(np.abs(o["phi"]).max(), 1e-300)
        assert np.abs(_np(g[f]) - o[f]).max() / s < 1e-10, f


@pytest.mark.parametrize("shape", [(33, 31), (45, 45), (47, 53), (63, 65)])
def test_forms_against_oracle(ctx, shape):
    """The right-hand sides of the other forms: the face-averaged balance
    (1e-10), the time-dependent one (1e-10) and the adjoint's (1e-9)."""
    nx, ny = shape
    p = inputs.random_problem(nx, ny, seed=6, sigma_range=(0.5, 5.0))
    _say("coarse cycle forms %s" % (shape,))
    kw = dict(synth_form=1, synth_sub=2)
    g = gsis.gsis_solve(ctx, p, tol=0.0, max_iter=3, synth_rtol=1e-15, synth_max_iter=200, **kw)
    o = oracle.solve(p, tol=0.0, max_iter=3, **kw)
    assert _rel(g["phi"], o["phi"]) < 1e-10
    rng = np.random.Generator(np.random.PCG64(nx))
    cv, T0 = rng.uniform(0.5, 2.0, nx * ny), rng.uniform(0.2, 1.2, nx * ny)
    mat = dict(c=2.0, a=0.7, dt=0.05, sub_iter=3)
    pl = gsis.TDPlan(ctx, p, T0, cv=cv, **mat, tol=0.0, max_iter=2, synth_rtol=1e-15,
                     synth_max_iter=300)
    pl.advance(2)
    t = pl.read_td()
    pl.close()
    o = oracle.td_solve(p, T0, 2, cv=cv, tol=0.0, max_iter=2, **mat)
    assert _rel(t["rho"], o["rho"]) < 1e-10 and _rel(t["T"], o["T"]) < 1e-10
    gphi = rng.uniform(-1.0, 1.0, nx * ny)
    pl = gsis.Plan(ctx, p, tol=1e-13, max_iter=3000, synth_rtol=1e-13, synth_max_iter=200,
                   limiter=0)
    pl.iterate(3000)
    ga, gs, gq, info = pl.adjoint(g_phi=gphi, tol=1e-13, max_iter=3000)
    pl.close()
    r = oracle.solve(p, tol=1e-14, max_iter=5000, limiter=0, return_I=True)
    o = oracle.adjoint(p, r["I"], gphi, tol=1e-14, limiter=0)
    assert _rel(ga, o["g_sigma_a"]) < 1e-9 and _rel(gs, o["g_sigma_s"]) < 1e-9
    assert _rel(gq, o["g_q"]) < 1e-9


@pytest.mark.parametrize("shape", [(9, 8), (33, 31), (45, 45), (63, 65)])
@pytest.mark.parametrize("cap", [4, 200])
def test_small_solve_is_the_batched_one(ctx, shape, cap):
    """The solve in one workgroup takes the iterations of the one in separate
    kernels (a batch with a grid that needs them), also where the cap ends it
    unconverged (at four: a batch takes no fewer): the same recurrence in
    another order of summation, 1e-10."""
    p = inputs.random_problem(shape[0], shape[1], seed=8, sigma_range=(0.5, 20.0))
    big = inputs.random_problem(70, 67, seed=9, sigma_range=(0.5, 20.0))
    _say("small solve %s cap %d" % (shape, cap))
    kw = dict(tol=0.0, max_iter=3, synth_rtol=1e-12, synth_max_iter=cap)
    s = gsis.gsis_solve(ctx, p, **kw)
    b = gsis.Batch(ctx, [p, big], **kw)
    b.iterate(3)
    r = b.read(0)
    b.close()
    assert _rel(s["phi"], _np(r["phi"])) < 1e-10
