"""Energies on the paths by Newton's third law with the series cut short
(mixed) or absent (the FP32 estimate): as accurate as the direct kernel's, which
sums q_j r^-1 with the same terms of the series.  Both take the same r^-1 of
every pair, so they agree to the rounding of sums of terms of one sign (2e-15;
r^-1 taken as r^2 r^-3 is off by 5.8e-15 and 1e-8 more)."""
import numpy as np
import pytest

from test_gpu_rows import _cloud, api  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = 2e-15
DIRECT = dict(p=1, wg=64, splits=16, algo=0)


def _forced(api, op, n, prec, call, **cfg):
    api.set_config(op, n, prec, **cfg)
    try:
        return call()
    finally:
        api.reset_config(op, n, prec)


def _inputs(n):
    from _gpu_util import dev
    st, q, m, trap = _cloud(n, n)
    return st, [dev(st[k]) for k in range(3)], q, dev(q), dev(m), trap


@pytest.mark.parametrize("one_charge", [False, True])
@pytest.mark.parametrize("prec", ["mixed", "fp32"])
@pytest.mark.parametrize("n", [6145, 9000, 12001, 16383])
def test_one_run(api, n, prec, one_charge):  # noqa: F811
    from _gpu_util import dev, state_tensors
    st, (x, y, z), q, qd, m, trap = _inputs(n)
    if one_charge:
        qd = dev(np.full(n, q[1]))
    for eps2 in (0.0, 1e-12):
        u = _forced(api, "energy", n, prec, lambda: api.coulomb_energy(x, y, z, qd, eps2, prec).item(), **DIRECT)
        assert abs(api.coulomb_energy(x, y, z, qd, eps2, prec).item() - u) <= TOL * u
        assert api.get_path("grad", n, prec) == "shares"
        g = api.coulomb_trap_grad(x, y, z, qd, eps2=eps2, prec=prec, energy=True)[1].item()
        assert abs(g - u) <= TOL * u
        rec = api.md_run(state_tensors(st), qd, m, trap, 0.0, 1e-9, 0, eps2=eps2, every=1, prec=prec)[0, 0, 1].item()
        assert abs(rec - u) <= TOL * u


@pytest.mark.parametrize("prec", ["mixed", "fp32"])
def test_ensemble(api, prec):  # noqa: F811
    from _gpu_util import dev, state_tensors
    sizes = [2048, 3000, 17, 4096, 255] * 4
    parts = [_cloud(n, 40 + r) for r, n in enumerate(sizes)]
    st = np.concatenate([p[0] for p in parts], axis=1)
    q, m = (dev(np.concatenate([p[k] for p in parts])) for k in (1, 2))
    offs = np.concatenate([[0], np.cumsum(sizes)])
    run = lambda: api.md_run(state_tensors(st), q, m, parts[0][3], 0.0, 1e-9, 0, offsets=offs, every=1,  # noqa: E731
                             prec=prec)[:, 0, 1].cpu().numpy()
    want = _forced(api, "md_ensemble", int(offs[-1]), prec, run, p=4, wg=512, splits=1, algo=0)
    assert np.all(np.abs(run() - want) <= TOL * want)


@pytest.mark.parametrize("prec", ["mixed", "fp32"])
def test_bands(api, prec):  # noqa: F811
    n = 262145
    _, (x, y, z), _, q, m, trap = _inputs(n)
    u = _forced(api, "energy", n, prec, lambda: api.coulomb_energy(x, y, z, q, 0.0, prec).item(), **DIRECT)
    assert api.get_path("energy", n, prec) == "bands"
    assert abs(api.coulomb_energy(x, y, z, q, 0.0, prec).item() - u) <= TOL * u
    g = api.coulomb_trap_grad(x, y, z, q, prec=prec, energy=True)[1].item()
    assert abs(g - u) <= TOL * u
