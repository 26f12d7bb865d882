"""GPU: GSIS with ordinates in parts (many ordinates on few tiles) and on
either side of the lines of that rule, against the oracle."""
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


@pytest.mark.parametrize("shape,quad", [((1, 1), (20, 40)), ((17, 19), (20, 40)),
                                        ((64, 32), (20, 40)), ((65, 32), (20, 40)),
                                        ((17, 19), (19, 42))])
def test_gsis_moments_against_oracle(ctx, shape, quad):
    """phi and F of the second iterate (1e-12 and 1e-11, the bounds of the
    whole sums against the same oracle), and a batch's to the bit."""
    p = inputs.random_problem(shape[0], shape[1], quad=inputs.quad_gl_product_full(*quad),
                              seed=7, sigma_range=(0.1, 20.0))
    print("GSIS moments %s %s" % (shape, quad), flush=True)
    sys.stdout.flush()
    g = gsis.gsis_solve(ctx, p, synth_rtol=1e-15, synth_max_iter=200, tol=0.0, max_iter=2)
    o = oracle.solve(p, tol=0.0, max_iter=2)
    for f, tol in (("phi", 1e-12), ("Fx", 1e-11), ("Fy", 1e-11)):
        s = max(np.abs(o["phi"]).max(), 1e-300)
        assert np.abs(np.asarray(g[f]) - o[f]).max() / s < tol, f
    kw = dict(synth_rtol=1e-12, synth_max_iter=4, tol=0.0, max_iter=2)
    a = gsis.gsis_solve(ctx, p, **kw)
    b = gsis.Batch(ctx, [p, p], **kw)
    b.iterate(2)
    r = b.read(1)
    b.close()
    for f in ("phi", "Fx", "Fy"):
        assert np.array_equal(np.asarray(a[f]), np.asarray(r[f])), f
