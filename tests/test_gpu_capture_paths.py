"""md_run captured in a HIP graph on every path that the other capture tests do
not take: of one run, the forced pair launch and epilogue, a launch per step,
equal shares and the resident launch; of ensembles, whole rows and equal shares.
Every replay equals the eager run bitwise, with eager work on other data (in
the same workspace) between the replays."""
import numpy as np
import pytest

from test_gpu_rows import _cloud, api  # noqa: F401

pytestmark = pytest.mark.gpu
DT = 1e-9


def _replays(run, other, st):
    """run(tensors) -> records; other(): eager work between the replays."""
    import torch
    from _gpu_util import state_tensors
    eager, static, s0 = state_tensors(st), state_tensors(st), torch.stack(state_tensors(st))
    want = run(eager).clone()
    run(static)  # workspace and symbols exist before the capture

    def restore():
        for k in range(9):
            static[k].copy_(s0[k])

    restore()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        en = run(static)
    for rep in range(4):
        restore()
        en.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(torch.stack(static), torch.stack(eager)), rep
        assert torch.equal(en, want), rep
        other()
        torch.cuda.synchronize()


# The pair launch and its epilogue (forced); the resident launch; a launch per
# step, of 4 ions per workgroup and of 8; shares of 4 ions per lane and of 8.
@pytest.mark.parametrize("n,nsteps,every,forced", [
    (1024, 39, 1, dict(p=1, wg=256, splits=64, algo=0)), (1024, 39, 3, None), (1024, 4, 1, None), (1800, 9, 2, None),
    (7000, 5, 1, None), (33500, 4, 2, None)])
def test_one_run(api, n, nsteps, every, forced):  # noqa: F811
    from _gpu_util import dev, state_tensors
    st, q, m, trap = _cloud(n, n)
    q, m = dev(q), dev(m)
    if forced:
        api.set_config("md_run", n, "fp64", **forced)
    try:
        assert api.get_path("md_run", n) == ("config" if forced else "rows" if n <= 6144 else "shares")
        _replays(lambda ts: api.md_run(ts, q, m, trap, 0.0, DT, nsteps, every=every),
                 lambda: api.md_run(state_tensors(_cloud(n, 5)[0]), q, m, trap, 0.0, DT, 3, every=1), st)
    finally:
        api.reset_config("md_run", n)


# Few and many chunks for either shape of a launch: rows of four waves and of
# one, shares whose chunks eight waves finish and two.
@pytest.mark.parametrize("sizes", [[64, 600, 1, 333], [256] * 40, [2048, 3000, 17] * 6, [512, 1024, 700] * 160],
                         ids=["rows4", "rows1", "shares8", "shares2"])
def test_ensemble(api, sizes):  # noqa: F811
    from _gpu_util import dev, state_tensors

    def make(seed, ns):
        parts = [_cloud(n, seed + r) for r, n in enumerate(ns)]
        return (np.concatenate([p[0] for p in parts], axis=1), *(dev(np.concatenate([p[k] for p in parts])) for k in (1, 2)),
                [dict(p[3], gamma=5e-21 * (r % 2)) for r, p in enumerate(parts)],
                [int(o) for o in np.concatenate([[0], np.cumsum(ns)])])

    st, q, m, traps, offs = make(7, sizes)
    ost, oq, om, otraps, ooffs = make(8000, sizes[::-1])
    _replays(lambda ts: api.md_run(ts, q, m, [dict(t) for t in traps], 0.0, DT, 6, offsets=list(offs), every=2),
             lambda: api.md_run(state_tensors(ost), oq, om, otraps, 0.0, DT, 2, offsets=ooffs, every=1), st)
