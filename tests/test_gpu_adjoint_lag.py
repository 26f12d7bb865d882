"""GPU: the adjoint's sweep at the sizes where its form changes (steps between
waves and of the loads ahead; one workgroup or several per ordinate): every
form does the same operations on a cell, so the gradients are the same bits."""
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


@pytest.mark.parametrize("shape,parts", [((7, 256), ("1", "2", "4")), ((6, 257), ("1", "2")),
                                         ((6, 514), ("1", "2", "4")), ((23, 1000), ("1", "2", "4"))])
def test_sweep_forms_agree(ctx, shape, parts, monkeypatch):
    nx, ny = shape
    p = inputs.random_problem(nx, ny, seed=12, sigma_range=(0.5, 5.0))
    g = np.random.Generator(np.random.PCG64(ny)).uniform(-1.0, 1.0, nx * ny)
    first = None
    for n in parts:
        monkeypatch.setenv("GSIS_CHAIN_PARTS", n)
        print("adjoint sweep %s parts %s" % (shape, n), flush=True)
        sys.stdout.flush()
        pl = gsis.Plan(ctx, p, tol=1e-6, max_iter=500, limiter=0)
        pl.iterate(500)
        r = pl.adjoint(g_phi=g, tol=1e-6, max_iter=500)
        pl.close()
        r = [np.array(a) for a in r[:3]]
        first = first or r
        for a, b in zip(r, first):
            np.testing.assert_array_equal(a, b)
