"""GPU: gsis_solve_noalloc on problems that fill its region to within what
the fastest form of a plan keeps beyond what the solve needs (one more moment
partial per part of the ordinates, a hand-over buffer for the adjoint's sweep):
they are solved, with the fields of gsis_solve to the bit."""
import sys

import numpy as np
import pytest

from paper_2507_03975_amd import gsis, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gsis.Context(0)


def _same(a, b):
    for k in ("phi", "Fx", "Fy", "err_hist"):
        assert np.array_equal(np.asarray(a[k]), np.asarray(b[k])), k
    # (the residual's norm is summed by tiles, whose length the lean form may
    # change)
    np.testing.assert_allclose(a["tres_hist"], b["tres_hist"], rtol=1e-12)
    assert a["n_iter"] == b["n_iter"] and a["status"] == b["status"]


# 80 x 80: 2400 ordinates in parts keep 9 MB of partials, 7 MB are left; the
# others: more than 128 rows, 0.1 to 0.3 MB left, less than a hand-over buffer
@pytest.mark.parametrize("nx,ny,quad", [(80, 80, (50, 48)), (262, 224, (10, 24)),
                                        (295, 240, (12, 16))])
@pytest.mark.parametrize("method", [gsis.GSIS_SI, gsis.GSIS_GSIS])
def test_problems_at_the_limit(ctx, nx, ny, quad, method):
    p = inputs.random_problem(nx, ny, quad=inputs.quad_gl_product_full(*quad), seed=1)
    print("noalloc limit %dx%d %s method %d" % (nx, ny, quad, method), flush=True)
    sys.stdout.flush()
    kw = dict(method=method, tol=0.0, max_iter=2, limiter=0)
    _same(gsis.gsis_solve(ctx, p, noalloc=True, **kw), gsis.gsis_solve(ctx, p, **kw))


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("kw", [dict(), dict(method=0), dict(precision=1)])
def test_warm_start_and_inflow(ctx, device, kw):
    """A warm start and boundary intensities, whose set-up uses arrays of the
    region that are not in use yet."""
    import torch
    p = inputs.random_problem(37, 53, quad=inputs.quad_product(2, 16), seed=2)
    rng = np.random.Generator(np.random.PCG64(3))
    I0 = rng.uniform(0.0, 1.0, (37 * 53, len(p["mu"])))
    if device:
        p = {k: (torch.from_numpy(v).cuda() if isinstance(v, np.ndarray) else v)
             for k, v in p.items()}
        I0 = torch.from_numpy(I0).cuda()
    print("noalloc warm start device=%s %s" % (device, kw), flush=True)
    a = gsis.gsis_solve(ctx, p, noalloc=True, tol=0.0, max_iter=3, I0=I0, **kw)
    b = gsis.gsis_solve(ctx, p, tol=0.0, max_iter=3, I0=I0, **kw)
    for k in ("phi", "Fx", "Fy", "err_hist", "tres_hist"):
        x, y = (np.asarray(v[k].cpu() if hasattr(v[k], "cpu") else v[k]) for v in (a, b))
        assert np.array_equal(x, y), k
