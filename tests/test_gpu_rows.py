"""The one-launch paths that evaluate whole rows per workgroup: md_run and
md_step of one small run, ensembles of small runs, and forces, energy and
gradient of small clouds, at the edges of their tiles (4 or 8 ions per
workgroup, blocks of 64 j's, the size where the shape changes) against the
oracle and against the launches that a forced configuration takes."""
import numpy as np
import pytest

from paper_2106_11143_amd import inputs

pytestmark = pytest.mark.gpu
E = inputs.E_CHARGE
M40 = inputs.MASS_40U


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_11143_amd import api as A
    A.lib()
    return A


def _cloud(n, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    trap = inputs.pseudo_trap(1.0e6, 0.9e6, 0.2e6)
    sig = inputs.crystal_sigma(max(n, 2), trap["wx"], trap["wy"], trap["wz"])
    st = np.zeros((9, n))
    st[:3] = g.normal(size=(3, n)) * sig[:, None]
    st[3:6] = inputs.maxwell(g, n, 10e-3, M40)
    st[6:9] = g.normal(size=(3, n)) * 1e9  # a_0 as given without CB_INIT_ACCEL
    q = np.full(n, E)
    q[::5] *= 2.0
    m = np.full(n, M40)
    m[::3] *= 1.1
    return st, q, m, trap


# tile edges, block edges, both sides of the change of shape and of the limit
SIZES = [1, 2, 3, 4, 5, 8, 9, 63, 64, 65, 129, 513, 1536, 1537, 6144]


@pytest.mark.parametrize("n", SIZES)
def test_forces_gradient_and_energy(api, oracle, n):
    """Per ion 1e-12 (FP64) and 1e-7 (mixed) of the force, as for the pair
    kernels, and for the bare FP32 estimate 2e-6 of the ion's pair forces
    (kappa); the energy and the gradient to the same shares of their scale."""
    import torch
    from _gpu_util import dev
    st, q, m, trap = _cloud(n, 70 + n)
    x, y, z = st[:3]
    for eps2 in (0.0, 1e-14):
        *ref, kappa = oracle.forces(x, y, z, q, eps2=eps2, kappa=True)
        ref = np.stack(ref)
        u_ref, _ = oracle.coulomb_energy(x, y, z, q, eps2=eps2)
        norm = np.linalg.norm(ref, axis=0)
        k = np.array(api.trap_k(trap))[:, None]
        for prec, tol in (("fp64", 1e-12), ("ieee", 1e-12), ("mixed", 1e-7), ("fp32", 2e-6)):
            args = [dev(a) for a in (x, y, z, q)]
            F = torch.stack(api.coulomb_forces(*args, eps2=eps2, prec=prec)).cpu().numpy()
            g, u = api.coulomb_trap_grad(*args, dev(m), trap, 0.0, eps2, prec, energy=True)
            g0, _ = api.coulomb_trap_grad(*args, eps2=eps2, prec=prec)
            uc = api.coulomb_energy(*args, eps2=eps2, prec=prec).item()
            g, g0, u = g.cpu().numpy(), g0.cpu().numpy(), u.item()
            if n == 1:
                assert np.all(F == 0.0) and uc == 0.0
            else:
                err = np.linalg.norm(F - ref, axis=0) / norm
                assert np.all(err <= tol * (kappa if prec == "fp32" else 1.0)), (prec, eps2)
                assert abs(uc - u_ref) <= tol * abs(u_ref), (prec, eps2)
            assert np.array_equal(g0, -F), (prec, eps2)
            G = m * k * st[:3] - ref
            assert np.abs(g - G).max() <= tol * max(np.abs(ref).max(), np.abs(m * k * st[:3]).max())
            ut = 0.5 * (m * (k * st[:3] ** 2).sum(0)).sum()
            assert abs(u - u_ref - ut) <= tol * (abs(u_ref) + ut)
    assert api.poll_flags() == 0


@pytest.mark.parametrize("n", SIZES)
def test_md_run(api, oracle, n):
    """One launch per step by default: odd and even step counts (the last
    drift always lands in the caller's arrays), with and without
    CB_INIT_ACCEL and records, against the two-launch step (forced) to
    rounding and, up to 1537 ions, against the oracle."""
    from _gpu_util import dev, state_host, state_tensors
    st, q, m, trap = _cloud(n, 170 + n)
    trap = dict(inputs.rf_trap(0.01, 0.3, 10e6, 0.2e6, phase=0.4), gamma=2e5 * M40)
    dt = 2e-9
    for nsteps, every, init in ((0, 1, True), (1, 0, False), (5, 1, True), (6, 2, True), (6, 0, False), (7, 3, False)):
        got = {}
        for path in ("rows", "two-launch"):
            if path == "two-launch":
                api.set_config("md_run", n, "fp64", p=1, wg=64, splits=max(1, min(16, n // 64)), algo=0)
            try:
                ts = state_tensors(st)
                en = api.md_run(ts, dev(q), dev(m), trap, 3e-8, dt, nsteps, every=every, init_accel=init)
                got[path] = (state_host(ts), en.cpu().numpy()[0] if every else np.zeros((1, 4)))
            finally:
                api.reset_config("md_run", n, "fp64")
        a, b = got["rows"], got["two-launch"]
        for blk in (slice(0, 3), slice(3, 6), slice(6, 9)):
            scale = np.abs(b[0][blk]).max()
            assert np.abs(a[0][blk] - b[0][blk]).max() <= 1e-12 * scale, (nsteps, every, init, blk)
        assert np.abs(a[1] - b[1]).max() <= 1e-12 * np.abs(b[1]).max(), (nsteps, every, init)
        if n <= 1537 and nsteps and init:
            ref, en_ref, _ = oracle.md_run(st, q, m, trap, 3e-8, dt, nsteps, every=every)
            for blk in (slice(0, 3), slice(3, 6), slice(6, 9)):
                assert np.abs(a[0][blk] - ref[blk]).max() <= 1e-11 * np.abs(ref[blk]).max(), (n, blk)
            if every:
                assert np.abs(a[1] - en_ref).max() <= 1e-11 * np.abs(en_ref).max()
    assert api.poll_flags() == 0


@pytest.mark.parametrize("sizes", [[1, 2, 3], [1, 7, 8, 9, 63, 64, 65, 200], [100] * 90, [1000, 5, 64, 300] * 12])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_ensemble(api, sizes, prec):
    """Ensembles of small runs by default, few chunks (four waves each) and
    many (one wave each), against the persistent kernel (forced), every trap
    kind, odd and even step counts, records and none."""
    from _gpu_util import dev
    parts = [_cloud(n, 300 + 7 * r) for r, n in enumerate(sizes)]
    st = np.concatenate([p[0] for p in parts], axis=1)
    q, m = (np.concatenate([p[k] for p in parts]) for k in (1, 2))
    base = parts[0][3]
    kinds = [base, inputs.ramp_trap(1.5e6, 0.6e6, 0.15e6, 0.0, 20e-9), inputs.rf_trap(0.0, 0.3, 10e6, 0.15e6),
             dict(base, gamma=5e5 * M40)]
    traps = [kinds[r % 4] for r in range(len(sizes))]
    offs = np.concatenate([[0], np.cumsum(sizes)])
    for nsteps, every, init in ((0, 1, True), (5, 2, True), (6, 3, False), (6, 0, True), (1, 0, False)):
        got = []
        for persistent in (False, True):
            if persistent:
                api.set_config("md_ensemble", offs[-1], prec, p=4, wg=512, splits=1, algo=0)
            try:
                ts = [dev(st[k]) for k in range(9)]
                en = api.md_run(ts, dev(q), dev(m), traps, 0.0, 1e-9, nsteps, offsets=offs, every=every, prec=prec,
                                init_accel=init)
                got.append((np.stack([t.cpu().numpy() for t in ts]), en.cpu().numpy() if every else np.zeros(1)))
            finally:
                api.reset_config("md_ensemble", offs[-1], prec)
        a, b = got
        for blk in (slice(0, 3), slice(3, 6), slice(6, 9)):
            assert np.abs(a[0][blk] - b[0][blk]).max() <= 1e-11 * np.abs(b[0][blk]).max(), (nsteps, every, init)
        assert np.abs(a[1] - b[1]).max() <= 1e-11 * max(np.abs(b[1]).max(), 1e-300), (nsteps, every, init)
    assert api.poll_flags() == 0


@pytest.mark.parametrize("n", [900, 2500, 9000])
def test_resumed_records_are_bitwise(api, n):
    """A record is summed by the next step's launch, or after the last step by
    one of its own: both in the same order, so a run resumed after a record
    agrees bitwise, state and records."""
    from _gpu_util import dev, state_host, state_tensors
    st, q, m, trap = _cloud(n, 11)
    q, m = dev(q), dev(m)
    a, b = state_tensors(st), state_tensors(st)
    ea = api.md_run(a, q, m, trap, 0.0, 1e-9, 6, every=2).cpu().numpy()
    eb = api.md_run(b, q, m, trap, 0.0, 1e-9, 4, every=2).cpu().numpy()
    ec = api.md_run(b, q, m, trap, 4e-9, 1e-9, 2, every=2, init_accel=False).cpu().numpy()
    assert np.array_equal(state_host(a), state_host(b))
    assert np.array_equal(ea[0, :3], eb[0]) and np.array_equal(ea[0, 2:], ec[0])
