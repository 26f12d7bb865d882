"""GPU: residual tiles of the shortest and the longest lengths, bit for bit
against tiles of 31 diagonals, in every form that has them: FP64 with each face
option, FP32-mixed, time-dependent and batches, on grids of one to three bands
of rows and of fewer and more diagonals than the longest tile."""
import sys

import numpy as np
import pytest

from paper_2507_03975_amd import gsis, inputs

pytestmark = pytest.mark.gpu
LENGTHS = ("31", "3", "7", "51", "55", "59")
SHAPES = [(40, 17), (61, 70), (150, 130), (70, 200)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gsis.Context(0)


def _prob(shape, seed=9):
    return inputs.random_problem(*shape, quad=inputs.quad_product(1, 8), seed=seed,
                                 sigma_range=(0.05, 50.0))


def _np(a):
    return a.cpu().numpy() if hasattr(a, "cpu") else np.asarray(a)


def _each(monkeypatch, what, run):
    monkeypatch.setenv("GSIS_SWEEP_REFERENCE", "0")
    ref = None
    for rd in LENGTHS:
        monkeypatch.setenv("GSIS_RESID_DIAGONALS", rd)
        print("residual tiles of %s: %s" % (rd, what), flush=True)
        sys.stdout.flush()
        out = [_np(a) for a in run()]
        ref = ref or out
        for a, b in zip(ref, out):
            assert np.array_equal(a, b), rd


@pytest.mark.parametrize("kw", [dict(order=1, limiter=0), dict(limiter=0), dict(limiter=1),
                                dict(limiter=1, precision=1), dict(limiter=0, precision=1)])
@pytest.mark.parametrize("shape", SHAPES)
def test_plans(ctx, shape, kw, monkeypatch):
    p = _prob(shape)

    def run():
        r = gsis.gsis_solve(ctx, p, tol=0.0, max_iter=3, method=gsis.GSIS_SI, **kw)
        return r["phi"], r["Fx"], r["Fy"]
    _each(monkeypatch, "%s %s" % (shape, kw), run)


@pytest.mark.parametrize("shape", SHAPES[1:3])
def test_time_steps(ctx, shape, monkeypatch):
    p = _prob(shape)
    rng = np.random.Generator(np.random.PCG64(3))
    T0 = rng.uniform(0.2, 1.2, shape[0] * shape[1])

    def run():
        pl = gsis.TDPlan(ctx, p, T0, cv=1.0, c=2.0, a=0.7, dt=0.05, sub_iter=2, method=0, tol=0.0,
                         max_iter=2)
        pl.advance(2)
        r = pl.read_td()
        pl.close()
        return r["rho"], r["T"], r["Fx"], r["Fy"]
    _each(monkeypatch, "time steps %s" % (shape,), run)


@pytest.mark.parametrize("precision", [0, 1])
def test_batch(ctx, precision, monkeypatch):
    probs = [_prob(s, 20 + i) for i, s in enumerate(SHAPES)]

    def run():
        b = gsis.Batch(ctx, probs, method=0, tol=0.0, max_iter=2, precision=precision)
        b.iterate(2)
        out = [b.read(i)[k] for i in range(len(probs)) for k in ("phi", "Fx", "Fy")]
        b.close()
        return out
    _each(monkeypatch, "batch precision %d" % precision, run)


@pytest.mark.parametrize("shape,quad", [((400, 450), (1, 4)), ((782, 5), (1, 1)), ((60, 70), (2, 8)),
                                        ((90, 100), (3, 8))])
def test_few_ordinates(ctx, shape, quad, monkeypatch):
    """The length chosen where the ordinates go to fewer than eight XCDs, or to
    some of them twice: the bits of 31 diagonals."""
    monkeypatch.setenv("GSIS_SWEEP_REFERENCE", "0")
    p = inputs.random_problem(*shape, quad=inputs.quad_product(*quad), seed=3,
                              sigma_range=(0.05, 50.0))
    out = []
    for rd in (None, "31"):
        if rd:
            monkeypatch.setenv("GSIS_RESID_DIAGONALS", rd)
        else:
            monkeypatch.delenv("GSIS_RESID_DIAGONALS", raising=False)
        print("chosen residual length %s %s" % (shape, quad), flush=True)
        out.append(gsis.gsis_solve(ctx, p, tol=0.0, max_iter=3, method=gsis.GSIS_SI))
    for k in ("phi", "Fx", "Fy"):
        assert np.array_equal(_np(out[0][k]), _np(out[1][k])), k
