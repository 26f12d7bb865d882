"""GPU: the number of workgroups that share an ordinate's recurrence, on
either side of the lines of its rule, and the same bits from all of them."""
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


@pytest.mark.parametrize("shape,precision,parts", [
    ((2000, 256), 0, 1), ((768, 257), 0, 1), ((769, 257), 0, 2), ((769, 257), 1, 1),
    ((769, 320), 0, 2), ((384, 321), 0, 1), ((385, 321), 0, 2), ((385, 384), 0, 2),
    ((385, 384), 1, 1), ((40, 385), 0, 2), ((40, 385), 1, 2)])
def test_parts_by_shape(ctx, shape, precision, parts, monkeypatch):
    monkeypatch.setenv("GSIS_SWEEP_REFERENCE", "0")
    p = inputs.random_problem(*shape, seed=3, sigma_range=(0.1, 5.0))
    print("chain parts %s precision %d" % (shape, precision), flush=True)
    sys.stdout.flush()
    out = []
    for force in (None, "1", "3"):
        if force is None:
            monkeypatch.delenv("GSIS_CHAIN_PARTS", raising=False)
        else:
            monkeypatch.setenv("GSIS_CHAIN_PARTS", force)
        pl = gsis.Plan(ctx, p, method=0, tol=0.0, max_iter=3, precision=precision)
        if force != "3":         # (fewer where three would leave one empty)
            assert pl.transport_form()[2] == (parts if force is None else 1)
        pl.iterate(3)
        out.append(pl.read())
        pl.close()
    for r in out[1:]:
        for k in ("phi", "Fx", "Fy"):
            assert np.array_equal(np.asarray(out[0][k]), np.asarray(r[k])), k
