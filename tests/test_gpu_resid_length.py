"""GPU: the residual kernel with the tile length chosen for the problem, over
the face options and sizes that reach its ends, bit for bit against tiles of
31 and 47 diagonals."""
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


@pytest.mark.parametrize("kw", [dict(order=1, limiter=0), dict(limiter=0), dict(limiter=1),
                                dict(limiter=1, precision=1)])
@pytest.mark.parametrize("shape,quad", [((1, 1), (1, 4)), ((3, 200), (1, 4)), ((200, 3), (1, 4)),
                                        ((32, 32), (2, 4)), ((130, 66), (2, 16)),
                                        ((256, 256), (4, 32))])
def test_chosen_length_bitwise(ctx, shape, quad, kw, monkeypatch):
    """Every cell-ordinate is formed from the same operands by the same
    operations wherever a tile begins, so phi and F do not depend on the
    length; the residual norm is summed per tile (1e-12)."""
    p = inputs.random_problem(*shape, quad=inputs.quad_product(*quad), seed=9,
                              sigma_range=(0.05, 50.0))
    print("residual length %s %s %s" % (shape, quad, kw), flush=True)
    sys.stdout.flush()
    monkeypatch.setenv("GSIS_SWEEP_REFERENCE", "0")
    out = []
    for rd in (None, "31", "47"):
        if rd is None:
            monkeypatch.delenv("GSIS_RESID_DIAGONALS", raising=False)
        else:
            monkeypatch.setenv("GSIS_RESID_DIAGONALS", rd)
        out.append(gsis.gsis_solve(ctx, p, tol=0.0, max_iter=3, method=gsis.GSIS_SI, **kw))
    for r in out[1:]:
        for k in ("phi", "Fx", "Fy"):
            assert np.array_equal(np.asarray(out[0][k]), np.asarray(r[k])), k
        np.testing.assert_allclose(out[0]["tres_hist"], r["tres_hist"], rtol=1e-12)
