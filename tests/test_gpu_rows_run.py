"""md_run of a small run, whose steps workgroups that stay resident take
together: bitwise the steps of one call each (which take one launch per step),
also when the launch gives up waiting and one workgroup takes the steps, on
several streams at once, and in a replayed graph.  Sizes at the edges of the
groups of 4 ions, the blocks of 64 j's and the shapes (256, 1280); numbers of
steps around a launch's 128 and the position ring's 8."""
import ctypes as C
import threading

import numpy as np
import pytest

from paper_2106_11143_amd import inputs
from test_gpu_rows import _cloud, api  # noqa: F401

pytestmark = pytest.mark.gpu
DT = 1e-9


def _trap(kind, trap):
    if kind == "rf":
        return inputs.rf_trap(0.01, 0.2, 20e6, 0.3e6)
    return dict(trap, gamma=5e-21) if kind == "damped" else trap


def _single_steps(api, st, q, m, trap, nsteps, every, prec):
    """The run as calls of one step: state, and the records at multiples of every."""
    from _gpu_util import state_tensors
    s, recs = state_tensors(st), []
    for k in range(nsteps):
        e = api.md_run(s, q, m, trap, k * DT, DT, 1, init_accel=k == 0, every=1, prec=prec).cpu().numpy()[0]
        if k == 0:
            recs.append(e[0])
        if (k + 1) % every == 0:
            recs.append(e[1])
    return s, np.array(recs)


@pytest.mark.parametrize("n,nsteps,every,kind,prec", [
    (9, 40, 1, "static", "fp64"), (63, 17, 5, "rf", "fp64"), (64, 8, 3, "damped", "mixed"),
    (150, 137, 10, "static", "fp64"), (256, 30, 1, "rf", "mixed"), (257, 30, 7, "static", "fp64"),
    (640, 12, 12, "damped", "ieee"), (1023, 20, 1, "static", "fp64"), (1280, 14, 4, "rf", "fp32")])
def test_bitwise_single_steps(api, n, nsteps, every, kind, prec):  # noqa: F811
    from _gpu_util import dev, state_host, state_tensors
    st, q, m, trap = _cloud(n, n)
    trap, q, m = _trap(kind, trap), dev(q), dev(m)
    ref, recs = _single_steps(api, st, q, m, trap, nsteps, every, prec)
    s = state_tensors(st)
    e = api.md_run(s, q, m, trap, 0.0, DT, nsteps, every=every, prec=prec).cpu().numpy()[0]
    t = state_tensors(st)
    api.md_run(t, q, m, trap, 0.0, DT, nsteps, prec=prec)  # no records
    if kind == "rf":
        # The time of a step rounds differently, t0 + k dt against k dt + dt: by
        # 1e-16 of it, which moves the drive (phase below 4) and what follows
        # from it by some 1e-15 of its size a step.
        a, b = state_host(s), state_host(ref)
        assert np.all(np.abs(a - b).max(axis=1) <= 1e-12 * np.abs(b).max(axis=1))
        np.testing.assert_allclose(e, recs, rtol=1e-12)
        assert np.array_equal(a, state_host(t))
    else:
        assert np.array_equal(state_host(s), state_host(ref))
        assert np.array_equal(state_host(t), state_host(ref))
        assert np.array_equal(e, recs)


@pytest.mark.parametrize("n,nsteps,every", [(10, 20, 0), (150, 137, 10), (700, 12, 1), (1280, 13, 0)])
def test_gives_up(api, n, nsteps, every):  # noqa: F811
    """No polls at all: the launch gives up, and its end takes the steps."""
    import torch
    from _gpu_util import dev, state_host, state_tensors
    st, q, m, trap = _cloud(n, n + 1)
    q, m = dev(q), dev(m)
    a, b = state_tensors(st), state_tensors(st)
    ea = api.md_run(a, q, m, trap, 0.0, DT, nsteps, init_accel=False, every=every)
    nrec = nsteps // every + 1 if every else 1
    eb = torch.zeros(nrec, 4, dtype=torch.float64, device="cuda")
    ws = torch.empty(api.workspace_size("md_run", n), dtype=torch.uint8, device="cuda")
    f = api.lib().cb_rows_run_spins
    f.argtypes = [C.c_int64, C.POINTER(api.State), C.c_void_p, C.c_void_p, C.POINTER(api.Trap), C.c_double, C.c_double,
                  C.c_int64, C.c_double, C.c_int32, C.c_void_p, C.c_int64, C.c_int32, C.c_void_p, C.c_size_t, C.c_void_p]
    tr, s = api.make_trap(trap), api._state(b)
    api._check(f(n, C.byref(s), q.data_ptr(), m.data_ptr(), C.byref(tr), 0.0, DT, nsteps, 0.0, 0,
                 eb.data_ptr() if every else None, every, 0, ws.data_ptr(), ws.numel(),
                 torch.cuda.current_stream().cuda_stream), "cb_rows_run_spins")
    assert np.array_equal(state_host(a), state_host(b))
    if every:
        assert np.array_equal(ea.cpu().numpy()[0, 1:], eb.cpu().numpy()[1:])


def test_streams(api):  # noqa: F811
    """More runs at once than are admitted together, each on its thread's stream."""
    import torch
    from _gpu_util import dev, state_host, state_tensors
    sizes = [1280, 150, 1000, 600, 1024, 300]
    jobs = []
    for k, n in enumerate(sizes):
        st, q, m, trap = _cloud(n, 50 + k)
        jobs.append((st, dev(q), dev(m), trap))
    want = []
    for st, q, m, trap in jobs:
        s = state_tensors(st)
        api.md_run(s, q, m, trap, 0.0, DT, 300)
        want.append(state_host(s))
    got, streams = [state_tensors(j[0]) for j in jobs], [torch.cuda.Stream() for _ in jobs]
    torch.cuda.synchronize()

    def work(k):
        with torch.cuda.stream(streams[k]):
            _, q, m, trap = jobs[k]
            api.md_run(got[k], q, m, trap, 0.0, DT, 300)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for k in range(len(jobs)):
        assert np.array_equal(state_host(got[k]), want[k]), sizes[k]


def test_graph(api):  # noqa: F811
    import torch
    from _gpu_util import dev, state_host, state_tensors
    st, q, m, trap = _cloud(200, 3)
    q, m = dev(q), dev(m)
    s, r = state_tensors(st), state_tensors(st)
    run = lambda x: api.md_run(x, q, m, trap, 0.0, DT, 30, init_accel=False)  # noqa: E731
    api.md_run(s, q, m, trap, 0.0, DT, 30)  # (workspace and symbols exist before the capture)
    api.md_run(r, q, m, trap, 0.0, DT, 30)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        api.md_run(state_tensors(st), q, m, trap, 0.0, DT, 30)  # this stream's workspace
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        run(s)
    for _ in range(4):
        g.replay()
        run(r)
        torch.cuda.synchronize()
        assert np.array_equal(state_host(s), state_host(r))
