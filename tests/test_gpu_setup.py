"""GPU: set-up of a plan on the device: the first offending entry of host and
device inputs, aggregates on the threshold of the coupling ratio, and restarts
that repeat bit for bit."""
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


def _dev(p):
    import torch
    return {k: (torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")
                if isinstance(v, np.ndarray) else v) for k, v in p.items()}


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("bad,want", [
    ([("sigma_a", 37, -1.0)], "sigma_a[37]"),
    ([("sigma_s", 11, np.inf), ("sigma_a", 40, np.nan)], "sigma_s[11]"),
    ([("q", 5, np.nan), ("sigma_s", 5, -1.0)], "sigma_s[5]"),
    ([("sigma_a", 8, 0.0), ("sigma_s", 8, 0.0)], "sigma_a[8] + sigma_s[8]"),
    ([("q", 62, np.inf)], "q[62]"),
    ([("bnd_in", (3, 7), np.nan), ("bnd_in", (9, 2), np.nan)], "bnd_in[3][7]"),
    ([("bnd_in", (0, 0), np.nan), ("q", 62, np.inf)], "q[62]"),
])
def test_first_offending_entry(ctx, device, bad, want):
    p = inputs.random_problem(9, 7, seed=2)
    for name, at, v in bad:
        p[name] = p[name].copy()
        p[name][at] = v
    print("bad entry %s device=%s" % (want, device), flush=True)
    with pytest.raises(gsis.GSISError) as e:
        gsis.Plan(ctx, _dev(p) if device else p)
    assert e.value.status == gsis.GSIS_E_INVALID_ARG and want in str(e.value)


@pytest.mark.parametrize("shape", [(64, 32), (32, 64), (65, 33), (300, 1), (1, 300)])
def test_aggregates_on_the_threshold(ctx, shape):
    """A uniform medium on cells of aspect ratio 2 couples four times as
    strongly one way as the other, the ratio at which aggregates change; lines
    have one direction only. The synthetic solves (rtol 1e-15) hide the
    preconditioner from the iterates (1e-10, as the other edge strips)."""
    p = inputs.homogeneous(shape[0], shape[1], sigma_t=5.0)
    print("threshold %s" % (shape,), flush=True)
    sys.stdout.flush()
    g = gsis.gsis_solve(ctx, p, tol=0.0, max_iter=2, synth_rtol=1e-15, synth_max_iter=200)
    o = oracle.solve(p, tol=0.0, max_iter=2)
    assert np.abs(g["phi"] - o["phi"]).max() < 1e-10 * np.abs(o["phi"]).max()


@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(method=0)])
@pytest.mark.parametrize("warm", [False, True])
def test_restart_repeats(ctx, kw, warm):
    """A restarted plan (host or device arrays, with or without a warm start)
    gives the bits of its first run; so does a batch."""
    p = inputs.random_problem(37, 41, seed=5)
    I0 = np.random.default_rng(1).uniform(0.0, 0.3, (37 * 41, len(p["mu"]))) if warm else None
    runs = []
    for q in (p, _dev(p)):
        i0 = I0
        if I0 is not None and q is not p:
            import torch
            i0 = torch.from_numpy(I0).to("cuda:0")
        pl = gsis.Plan(ctx, q, I0=i0, tol=1e-9, max_iter=50, **kw)
        for _ in range(2):
            pl.reset()
            pl.iterate(5)
            r = pl.read()
            runs.append([np.asarray(r[k].cpu() if q is not p else r[k])
                         for k in ("phi", "Fx", "Fy", "err_hist", "tres_hist")])
        pl.close()
    if not warm:
        b = gsis.Batch(ctx, [p, p], tol=1e-9, max_iter=50, **kw)
        for _ in range(2):
            b.reset()
            b.iterate(5)
            r = [b.read(i) for i in (0, 1)]
            assert all(np.array_equal(r[0][k], r[1][k]) for k in ("phi", "Fx", "Fy"))
            runs.append([r[0][k] for k in ("phi", "Fx", "Fy", "err_hist", "tres_hist")])
        assert all(np.array_equal(x, y) for x, y in zip(runs[-1], runs[-2]))
        runs = runs[:-2]
        b.close()
    for r in runs[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(runs[0], r))
