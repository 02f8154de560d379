"""Middle sizes take equal shares of the Newton's-third-law pairs by default:
forces, energy, gradient and md_run at the edges of its blocks (256 or 512
ions), units (16 j's) and changes of shape, for three species layouts, against
the direct kernel (forced; the other tests tie it to the oracle) and, for one
size, the oracle."""
import numpy as np
import pytest

from paper_2106_11143_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2106_11143_amd import api as A
    A.lib()
    return A


def _ions(n, layout, seed):
    d = inputs.cloud100k(n=n, seed=seed)
    if layout == "uniform":
        d["q"][:] = inputs.E_CHARGE
    return inputs.group_by_charge(d) if layout == "grouped" else d


def _direct(api, n, prec, on):
    for op in ("forces", "energy", "md_run"):
        if on:
            api.set_config(op, n, prec, p=1, wg=256, splits=16, algo=0)
        else:
            api.reset_config(op, n, prec)


# either side of a block, of a unit and of each change of shape or path
SIZES = [6145, 6400, 6401, 6413, 12001, 17999, 18000, 27999, 28000, 28161, 57344]


@pytest.mark.parametrize("n,layout", [(n, ("uniform", "grouped", "random")[k % 3]) for k, n in enumerate(SIZES)])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_shares_match_the_direct_kernel(api, n, layout, prec):
    import torch
    from _gpu_util import dev
    d = _ions(n, layout, n)
    x, y, z, q, m = (dev(d[k]) for k in ("x", "y", "z", "q", "m"))
    st = inputs.state9(d)
    got = []
    for direct in (False, True):
        _direct(api, n, prec, direct)
        try:
            F = torch.stack(api.coulomb_forces(x, y, z, q, prec=prec))
            G, U = api.coulomb_trap_grad(x, y, z, q, m, d["trap"], prec=prec, energy=True)
            G0, _ = api.coulomb_trap_grad(x, y, z, q, prec=prec)
            uc = api.coulomb_energy(x, y, z, q, prec=prec)
            runs = []
            for nsteps, every, init in ((3, 2, True), (2, 0, False), (0, 1, True)):
                ts = [dev(st[k]) for k in range(9)]
                en = api.md_run(ts, q, m, d["trap"], 0.0, 1e-9, nsteps, every=every, init_accel=init, prec=prec)
                runs.append((torch.stack(ts), en))
            got.append((F, G, G0, U, uc, runs))
        finally:
            _direct(api, n, prec, False)
    tol = 1e-12 if prec == "fp64" else 1e-7
    (F, G, G0, U, uc, runs), (F1, G1, G01, U1, uc1, runs1) = got
    rel = torch.linalg.norm(F - F1, dim=0) / torch.linalg.norm(F1, dim=0)
    assert rel.max().item() <= tol
    assert torch.equal(G0, -F)
    assert (G - G1).abs().max().item() <= tol * G1.abs().max().item()
    assert abs((U - U1).item()) <= tol * abs(U1.item()) and abs((uc - uc1).item()) <= tol * abs(uc1.item())
    for (S, en), (S1, en1) in zip(runs, runs1):
        for b in (slice(0, 3), slice(3, 6), slice(6, 9)):
            assert (S[b] - S1[b]).abs().max().item() <= tol * S1[b].abs().max().item()
        if en is not None:
            assert (en - en1).abs().max().item() <= tol * en1.abs().max().item()
    assert torch.equal(torch.stack(api.coulomb_forces(x, y, z, q, prec=prec)), F)  # repeats bit for bit
    assert api.poll_flags() == 0


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("ieee", 1e-12), ("mixed", 1e-7), ("fp32", 2e-6)])
def test_shares_match_the_oracle(api, oracle, prec, tol):
    from _gpu_util import dev
    n = 7001
    for eps2 in (0.0, 1e-12):
        d = _ions(n, "random", 5)
        *ref, kappa = oracle.forces(d["x"], d["y"], d["z"], d["q"], eps2=eps2, kappa=True)
        ref = np.stack(ref)
        F = np.stack([t.cpu().numpy() for t in api.coulomb_forces(*(dev(d[k]) for k in "xyzq"), eps2=eps2, prec=prec)])
        err = np.linalg.norm(F - ref, axis=0) / np.linalg.norm(ref, axis=0)
        assert np.all(err <= tol * (kappa if prec == "fp32" else 1.0))


def test_shares_carry_non_finite_values(api):
    """Coincident ions and a non-finite charge reach the forces and the flag,
    on the diagonal and off it."""
    from _gpu_util import dev
    n = 6500
    for i, j in ((10, 40), (10, 6000)):
        d = _ions(n, "uniform", 9)
        for c in "xyz":
            d[c][j] = d[c][i]
        F = np.stack([t.cpu().numpy() for t in api.coulomb_forces(*(dev(d[k]) for k in "xyzq"))])
        bad = ~np.isfinite(F).all(axis=0)
        assert sorted(np.flatnonzero(bad)) == [i, j]
        assert api.poll_flags() == 1
    d = _ions(n, "uniform", 9)
    d["q"][3000] = np.inf
    F = np.stack([t.cpu().numpy() for t in api.coulomb_forces(*(dev(d[k]) for k in "xyzq"))])
    assert not np.isfinite(F).any()
    assert api.poll_flags() == 1
