"""GPU: the adjoint on grids at the lines where the number of workgroups of
its sweep changes, bit for bit against a sweep in one."""
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


@pytest.mark.parametrize("shape", [(30, 128), (512, 129), (513, 129), (512, 192), (224, 193),
                                   (225, 193), (160, 257), (161, 257), (128, 513), (129, 513)])
def test_parts_of_the_sweep(ctx, shape, monkeypatch):
    p = inputs.random_problem(*shape, seed=5, sigma_range=(0.5, 5.0))
    print("adjoint parts %s" % (shape,), flush=True)
    sys.stdout.flush()
    out = []
    for force in (None, "1"):
        if force is None:
            monkeypatch.delenv("GSIS_CHAIN_PARTS", raising=False)
        else:
            monkeypatch.setenv("GSIS_CHAIN_PARTS", force)
        pl = gsis.Plan(ctx, p, method=0, tol=1e-2, max_iter=300, limiter=0)
        pl.iterate(300)
        assert pl.status()[1] == 1
        out.append(pl.adjoint(p["sigma_a"], tol=0.0, max_iter=6))
        pl.close()
    for a, b in zip(out[0][:3], out[1][:3]):
        assert np.array_equal(np.asarray(a), np.asarray(b))
