"""GPU: the moments of small grids with many ordinates, whose quadrants are
summed in parts, against the oracle at the sizes where the division changes
(one tile, ragged tiles, the last grid that is divided, ordinates that do not
fill the last part)."""
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


@pytest.mark.parametrize("shape,quad", [((1, 1), (14, 16)), ((16, 16), (18, 24)),
                                        ((17, 33), (18, 24)), ((112, 64), (10, 20)),
                                        ((96, 80), (10, 20))])
@pytest.mark.parametrize("method", [gsis.GSIS_SI, gsis.GSIS_GSIS])
def test_divided_moments_against_oracle(ctx, shape, quad, method):
    """phi and F of a fixed iterate: a quadrant's sum of 50 to 108 terms in
    another order differs by a few ulps of its largest term (1e-12 and 1e-11,
    the tolerances of the undivided sums against the same oracle)."""
    p = inputs.random_problem(shape[0], shape[1], quad=inputs.quad_gl_product_full(*quad),
                              seed=7, sigma_range=(0.1, 20.0))
    print("moments %s %s method %d" % (shape, quad, method), flush=True)
    sys.stdout.flush()
    kw = dict(tol=0.0, max_iter=2, method=method)
    g = gsis.gsis_solve(ctx, p, synth_rtol=1e-15, synth_max_iter=200, **kw)
    o = oracle.solve(p, **kw)
    for f, tol in (("phi", 1e-12), ("Fx", 1e-11), ("Fy", 1e-11)):
        s = max(np.abs(o["phi"]).max(), 1e-300)
        assert np.abs(np.asarray(g[f]) - o[f]).max() / s < tol, f
