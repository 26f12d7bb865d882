"""GPU: arrays given as device memory that a kernel on the plan's device
cannot reach (pageable host memory), and arrays that it can (pinned host
memory), through the C-ABI with device_ptrs set. They go through the runtime's
copies, which write to pageable memory and refuse to read it: an error that
names the array, and the next call is none the worse. What is accepted gives the
fields of a plan of host arrays to the bit."""
import ctypes
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


@pytest.mark.parametrize("pinned", [True, False])
@pytest.mark.parametrize("where", ["bnd_in", "sigma_a", "outputs"])
def test_host_memory_among_device_arrays(ctx, where, pinned):
    import torch
    p = inputs.random_problem(37, 29, seed=4)
    print("host memory (pinned %s) as %s" % (pinned, where), flush=True)
    sys.stdout.flush()
    kw = dict(tol=0.0, max_iter=3)
    ref = gsis.gsis_solve(ctx, p, **kw)
    dev = {k: (torch.from_numpy(v).cuda() if isinstance(v, np.ndarray) else v)
           for k, v in p.items()}
    lib = gsis.load()
    a = gsis._Args(dev)
    o = gsis.make_options(**kw)
    o.device_ptrs = 1
    o.stream = torch.cuda.current_stream().cuda_stream
    (phi, fx, fy, hist, thist), r = gsis._result_buffers(a, 3)

    def host(n):
        return torch.empty(n, dtype=torch.float64, pin_memory=pinned)
    if where != "outputs":
        b = host(p[where].size)
        b.copy_(torch.from_numpy(p[where].ravel()))
        setattr(a.s, where, b.data_ptr())
        out = (phi, fx, fy, hist, thist)
    else:
        out = tuple(host(t.numel()).zero_() for t in (phi, fx, fy, hist, thist))
        r = gsis.gsis_result(*[t.data_ptr() for t in out], 0, 0.0)
    st = lib.gsis_solve(ctx.handle, ctypes.byref(a.s), ctypes.byref(o), ctypes.byref(r))
    if where != "outputs" and not pinned:
        assert st == gsis.GSIS_E_DEVICE and where in gsis.gsis_last_error(ctx)
        r = gsis.gsis_solve(ctx, dev, **kw)
        assert np.array_equal(r["phi"].cpu().numpy(), np.asarray(ref["phi"]))
        return
    assert st in (gsis.GSIS_OK, gsis.GSIS_NOT_CONVERGED), gsis.gsis_last_error(ctx)
    assert r.n_iter == 3
    for t, k in zip(out, ("phi", "Fx", "Fy", "err_hist", "tres_hist")):
        assert np.array_equal(t.cpu().numpy(), np.asarray(ref[k])), k
