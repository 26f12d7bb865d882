"""GPU: a problem's phi and F in a batch are those of its own plan, to the bit:
with problems on either side of the sizes whose synthetic solve is one kernel,
with small problems that share that kernel with larger ones, with ordinates that
a plan sums in parts, and whichever problems have left the batch."""
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


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _same(a, b, what):
    for k in ("phi", "Fx", "Fy"):
        x, y = (np.asarray(v[k].cpu() if hasattr(v[k], "cpu") else v[k]) for v in (a, b))
        assert np.array_equal(x, y), (what, k)


def _prob(nx, ny, seed, quad=None):
    return inputs.random_problem(nx, ny, quad=quad, seed=seed, sigma_range=(0.1, 20.0))


# at most 1024, 2048, 3072 and 4096 cells: one to four pairs of cells a thread
SMALL = [(1, 1), (9, 8), (33, 31), (45, 45), (47, 53), (63, 65), (64, 64)]
LARGE = [(70, 67), (130, 90)]


@pytest.mark.parametrize("which", ["mixed", "small", "few"])
@pytest.mark.parametrize("kw", [dict(method=0), dict(limiter=0), dict(precision=1)])
def test_batch_is_alone(ctx, which, kw):
    """The cap on the CG iterations (four, which a batch also takes) ends
    every solve alike in both."""
    many = inputs.quad_gl_product_full(18, 24)
    probs = [_prob(nx, ny, 3 + i) for i, (nx, ny) in enumerate(SMALL)]
    probs.append(_prob(17, 33, 40, many))
    if which == "mixed":
        probs += [_prob(nx, ny, 50 + i) for i, (nx, ny) in enumerate(LARGE)]
    if which == "few":
        probs = [probs[1], probs[7]]
    _say("batch %s %s" % (which, kw))
    opt = dict(tol=0.0, max_iter=3, synth_rtol=1e-12, synth_max_iter=4, **kw)
    b = gsis.Batch(ctx, probs, **opt)
    b.iterate(3)
    for i, p in enumerate(probs):
        _same(gsis.gsis_solve(ctx, p, **opt), b.read(i), (p["nx"], p["ny"]))
    b.close()


@pytest.mark.parametrize("ask", [1, 4, 40])
def test_numbers_do_not_depend_on_who_is_left(ctx, ask):
    """A large, almost absorbing problem converges first. Asking for the status
    takes it out of the batch; the small ones' numbers stay those of their own
    plans."""
    big = inputs.random_problem(90, 80, seed=2, sigma_range=(5.0, 9.0), c_range=(0.0, 0.05))
    probs = [_prob(33, 31, 6), big, _prob(64, 64, 8)]
    opt = dict(tol=1e-7, max_iter=200, limiter=0, synth_rtol=1e-12, synth_max_iter=4)
    _say("who is left, status every %d" % ask)
    b = gsis.Batch(ctx, probs, **opt)
    n = 0
    while n < 200:
        b.iterate(ask)
        n += ask
        if b.status()[3] == len(probs):
            break
    for i, p in enumerate(probs):
        s, r = gsis.gsis_solve(ctx, p, **opt), b.read(i)
        assert s["n_iter"] == r["n_iter"], i
        _same(s, r, i)
    b.close()
