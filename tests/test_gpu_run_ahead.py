"""GPU: plans whose synthetic solve is one kernel enqueue iterations without
waiting for each, but never more than 16 past the end of a solve of eight or more, in one call
or over many, and start anew after a reset."""
import sys

import numpy as np
import pytest

from paper_2507_03975_amd import gsis, inputs

pytestmark = pytest.mark.gpu
AHEAD = 16


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gsis.Context(0)


@pytest.mark.parametrize("step", [1, 7, 8, 1000])
def test_iterations_past_the_end(ctx, step):
    """The phase timer counts the iterations that were enqueued."""
    p = inputs.random_problem(24, 19, seed=1, sigma_range=(0.5, 5.0))
    print("run ahead, calls of %d" % step, flush=True)
    sys.stdout.flush()
    pl = gsis.Plan(ctx, p, tol=1e-8, max_iter=500, limiter=0, profile=1)
    out = []
    for _ in range(2):
        for _ in range(0, 1000, step):
            pl.iterate(step)
        n, conv, _ = pl.status()
        assert conv == 1 and n > AHEAD // 2
        enqueued = pl.phase_times()[1]
        assert n <= enqueued <= n + AHEAD, (n, enqueued)
        pl.iterate(5)                 # past the end: nothing to do
        out.append(pl.read())
        assert pl.status()[0] == n
        pl.reset()
        pl.phase_times()
    pl.close()
    for k in ("phi", "Fx", "Fy", "err_hist"):
        assert np.array_equal(np.asarray(out[0][k]), np.asarray(out[1][k])), k
