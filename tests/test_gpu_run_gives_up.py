"""Small runs whose resident launch gives up, or is not admitted at all: the
words in the workspace that say so, the same results bit for bit, and about the
time of a launch per step (a run that shares the GPU must not become a run on
one of its compute units)."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_rows import _cloud, api  # noqa: F401

pytestmark = pytest.mark.gpu
DT = 1e-9
NORMAL = 1 << 18


def _hook(api):
    f = api.lib().cb_rows_run_spins
    f.argtypes = [C.c_int64, C.POINTER(api.State), C.c_void_p, C.c_void_p, C.POINTER(api.Trap), C.c_double, C.c_double,
                  C.c_int64, C.c_double, C.c_int32, C.c_void_p, C.c_int64, C.c_int32, C.c_void_p, C.c_size_t, C.c_void_p]
    return f


def _run(api, f, ts, q, m, trap, nsteps, every, prec, spins, en=None, ws=None):
    import torch
    n = q.numel()
    ws = torch.zeros(api.workspace_size("md_run", n), dtype=torch.uint8, device="cuda") if ws is None else ws
    tr, s = api.make_trap(trap), api._state(ts)
    api._check(f(n, C.byref(s), q.data_ptr(), m.data_ptr(), C.byref(tr), 0.0, DT, nsteps, 0.0, api._prec(prec),
                 en.data_ptr() if every else None, every, spins, ws.data_ptr(), ws.numel(),
                 torch.cuda.current_stream().cuda_stream), "cb_rows_run_spins")
    return ws


# The edges of the groups of 4 ions and of the shapes (256, 1280); runs of one
# launch and of several, whose last is short; every trap kind's friction branch.
@pytest.mark.parametrize("n,nsteps,every,gamma,prec", [
    (10, 20, 0, 0.0, "fp64"), (150, 137, 10, 0.0, "fp64"), (256, 128, 128, 5e-21, "mixed"), (257, 129, 1, 0.0, "ieee"),
    (700, 12, 1, 5e-21, "fp64"), (1023, 140, 7, 0.0, "fp32"), (1280, 13, 0, 0.0, "fp64")])
@pytest.mark.parametrize("spins", [0, -1])
def test_same_bits_and_says_so(api, n, nsteps, every, gamma, prec, spins):  # noqa: F811
    import torch
    from _gpu_util import dev, state_host, state_tensors
    st, q, m, trap = _cloud(n, n + 1)
    trap, q, m = dict(trap, gamma=gamma), dev(q), dev(m)
    f = _hook(api)
    nrec = nsteps // every + 1 if every else 1
    got = {}
    for k in (NORMAL, spins):
        ts = state_tensors(st)
        en = torch.zeros(nrec, 4, dtype=torch.float64, device="cuda")
        ws = _run(api, f, ts, q, m, trap, nsteps, every, prec, k, en)
        word = ws[:8].view(torch.int32).cpu().numpy()
        waves = (n + 3) // 4 * (4 if n <= 256 else 8)
        assert tuple(word) == ((0, waves) if k == NORMAL else (1, waves if k == 0 else 0))
        got[k] = state_host(ts), en.cpu().numpy()
    assert np.array_equal(got[NORMAL][0], got[spins][0])
    assert np.array_equal(got[NORMAL][1], got[spins][1])
    assert api.poll_flags() == 0


@pytest.mark.parametrize("n", [150, 1024, 1280])
def test_costs_about_a_launch_per_step(api, n):  # noqa: F811
    """Within five times the steps as calls of four (a launch each): by one
    workgroup they took 9 to 117 times as long."""
    import torch
    from _gpu_util import dev, state_tensors
    st, q, m, trap = _cloud(n, n)
    q, m, ts = dev(q), dev(m), state_tensors(st)
    f = _hook(api)
    ws = torch.zeros(api.workspace_size("md_run", n), dtype=torch.uint8, device="cuda")

    def steps():
        for _ in range(32):
            api.md_run(ts, q, m, trap, 0.0, DT, 4, init_accel=False)

    def ms(call):
        call()
        t = []
        for _ in range(3):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            call()
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
        return min(t)

    single = ms(steps)
    for spins in (0, -1):
        gave_up = ms(lambda: _run(api, f, ts, q, m, trap, 128, 0, "fp64", spins, ws=ws))
        print(f"[n={n}] 128 steps, a launch each {1e3 * single:.0f} us, given up (spins {spins}) {1e3 * gave_up:.0f} us",
              flush=True)
        assert gave_up <= 5 * single
