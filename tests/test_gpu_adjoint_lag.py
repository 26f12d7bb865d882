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


@pytest.mark.parametrize("shape", [(63, 64), (64, 64), (65, 130), (130, 65)])
@pytest.mark.parametrize("order", [1, 2])
def test_cells_of_a_diagonal_against_oracle(ctx, shape, order):
    """The transposed residual takes neighbours from other lanes where a
    wave's 64 cells lie on one diagonal: the first grids that have such waves,
    whole and ragged. Both sides stop at relative changes of 1e-12 or less,
    contracting by 0.8 to 0.9 a pass, so they differ by some 1e-11 of the
    iterates and up to 1e3 times that of the gradients: 1e-8 (a wrong neighbour
    is an error of order one)."""
    import oracle
    nx, ny = shape
    p = inputs.random_problem(nx, ny, seed=4, sigma_range=(0.5, 5.0))
    g = np.random.Generator(np.random.PCG64(nx)).uniform(-1.0, 1.0, nx * ny)
    print("adjoint diagonals %s order %d" % (shape, order), flush=True)
    sys.stdout.flush()
    kw = dict(limiter=0, order=order)
    pl = gsis.Plan(ctx, p, tol=1e-13, max_iter=3000, synth_rtol=1e-13, synth_max_iter=200, **kw)
    pl.iterate(3000)
    r = pl.adjoint(g_phi=g, tol=1e-12, max_iter=3000)
    pl.close()
    f = oracle.solve(p, tol=1e-13, max_iter=5000, return_I=True, **kw)
    o = oracle.adjoint(p, f["I"], g, tol=1e-12, max_iter=5000, **kw)
    for a, k in zip(r[:3], ("g_sigma_a", "g_sigma_s", "g_q")):
        assert np.abs(np.array(a) - o[k]).max() / np.abs(o[k]).max() < 1e-8, k
