"""GPU: time steps on grids with more source tiles than the chip starts at
once. The source that an iteration's end writes is what the next time step
begins with, also after the iteration that ended the step before: every tile
of it has to be of that iteration, however late its workgroup starts."""
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


def _rel(a, b):
    a = a.cpu().numpy() if hasattr(a, "cpu") else np.asarray(a)
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("shape", [(56000, 1), (1, 56000)])
def test_every_tile_of_a_steps_last_source(ctx, shape, method):
    """Three steps of two inner iterations, each step ended by the cap, on
    3500 tiles (some 2000 workgroups of the kernel run at once): to 1e-12 (SI)
    and 1e-10 (GSIS), the FP64 bounds of iterates."""
    N = shape[0] * shape[1]
    # (cells of unit size: the synthetic operator's condition stays small)
    p = dict(inputs.random_problem(*shape, seed=4, sigma_range=(0.5, 5.0)), dx=1.0, dy=1.0)
    rng = np.random.Generator(np.random.PCG64(N))
    cv, T0 = rng.uniform(0.5, 2.0, N), rng.uniform(0.2, 1.2, N)
    mat = dict(c=2.0, a=0.7, dt=0.05, sub_iter=2)
    print("td many tiles %s method=%d" % (shape, method), flush=True)
    sys.stdout.flush()
    pl = gsis.TDPlan(ctx, p, T0, cv=cv, **mat, method=method, tol=0.0, max_iter=2,
                     synth_rtol=1e-15, synth_max_iter=300)
    st, its, errs = pl.advance(3)
    g = pl.read_td()
    pl.close()
    o = oracle.td_solve(p, T0, 3, cv=cv, tol=0.0, max_iter=2, method=method, **mat)
    assert its == [2, 2, 2] == o["inner_iters"]
    tol = 1e-12 if method == 0 else 1e-10
    for k in ("rho", "T"):
        assert _rel(g[k], o[k]) < tol, k
    assert _rel(g["Fx"], o["Fx"]) < 10 * tol and _rel(g["Fy"], o["Fy"]) < 10 * tol
