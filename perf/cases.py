"""The work that a user of this framework has it do, as cases that can be timed.

Every case goes through the public Python entry points (``api``, ``autograd``,
``drivers``), which marshal arguments for the C ABI.  Units are SI and every
array is float64, as the library takes them.  A case is a dict of plain values:

- kind "md":       one trajectory, continued chunk by chunk (``api.md_run``
                   with the accelerations carried over, as a program does that
                   stores or prints something between chunks);
- kind "ensemble": many independent runs of uneven size in one ``api.md_run``;
- kind "forces":   one evaluation of the forces (``api.coulomb_forces``);
- kind "grad":     gradient and energy of the Coulomb and trap potential
                   (``api.coulomb_trap_grad``), one step of a minimiser;
- kind "hvp":      Hessian products with a block of vectors
                   (``api.coulomb_hvp``), one block of a normal-mode search;
- kind "autograd": energy, its gradient and a Hessian product through
                   ``torch.autograd`` (forward, backward, double backward);
- kind "traj":     d(mean-square displacement)/d(trap frequencies) by the
                   discrete adjoint (``drivers.traj_grad``).

``exact`` evaluates the same formulas in plain torch float64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2106_11143_amd import api, autograd, drivers, inputs

DEV = "cuda"


def listed():
    return [
        # A small trapped crystal, the size of most experiments: thousands of
        # steps follow each other and only their latency counts.
        dict(name="md_150", kind="md", n=150, cloud="gauss", trap="static", nsteps=100, every=10, prec="fp64"),
        # The 1024-ion cloud with its energies recorded at every step.
        dict(name="md_1024", kind="md", n=1024, cloud="gauss", trap="static", nsteps=100, every=1, prec="fp64"),
        # Statistics over a modest ensemble of small runs of uneven size.
        dict(name="ensemble_64", kind="ensemble", nrun=64, nmin=64, nmax=1024, nsteps=50, every=25, prec="fp64"),
        # 32768 ions under the explicit RF drive, no records.
        dict(name="md_rf_32768", kind="md", n=32768, cloud="ellipsoid", trap="rf", nsteps=5, every=0, prec="fp64"),
        # The headline: 1e5 ions, 1% doubly charged, ions of one charge contiguous.
        dict(name="md_100000", kind="md", n=100000, cloud="two_species_grouped", trap="static", nsteps=2, every=0,
             prec="fp64"),
        # One force evaluation between the small and the large sizes, ragged,
        # on the mixed-precision path.
        dict(name="forces_12001_mixed", kind="forces", n=12001, cloud="gauss", prec="mixed"),
        # The largest: three times the headline's ions in the seeded order
        # (species interleaved).
        dict(name="forces_300001", kind="forces", n=300001, cloud="two_species", prec="fp64"),
        # A minimiser's step on a large two-species cloud: gradient and energy.
        dict(name="grad_65537", kind="grad", n=65537, cloud="two_species", trap="static", prec="fp64"),
        # A block of the normal-mode search on 8192 ions.
        dict(name="hvp_8192x8", kind="hvp", n=8192, nvec=8, cloud="crystal", trap="static", prec="fp64"),
        # Energy, gradient and Hessian product of a small cloud by autograd.
        dict(name="autograd_1000", kind="autograd", n=1000, cloud="gauss", trap="static", prec="fp64"),
        # The trajectory gradient at the crystal's size, fewer steps.
        dict(name="traj_8192", kind="traj", n=8192, cloud="crystal", nsteps=20, checkpoint=10, prec="fp64"),
        # The Kibble-Zurek ensemble: 512 runs of 64 to 4096 ions.
        dict(name="ensemble_512", kind="ensemble", nrun=512, nmin=64, nmax=4096, nsteps=10, every=0, prec="fp64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["md", "md", "md", "ensemble", "ensemble", "forces", "forces", "grad", "hvp", "autograd", "traj"])
    prec = rng.choice(["fp64", "fp64", "fp64", "mixed"])
    if kind == "md":
        n = _log_int(rng, 16, 100000)
        most = 100 if n <= 4096 else (20 if n <= 32768 else 4)
        return dict(kind="md", n=n, cloud=rng.choice(["gauss", "ellipsoid", "two_species", "two_species_grouped"]),
                    trap=rng.choice(["static", "rf", "damped"]), nsteps=rng.randint(2, most),
                    every=rng.choice([0, 0, 1, 5]), prec=prec)
    if kind == "ensemble":
        nmax = _log_int(rng, 100, 4096)
        nrun = _log_int(rng, 2, 512)
        most = 50 if nrun * nmax * nmax < 3e8 else 10
        return dict(kind="ensemble", nrun=nrun, nmin=min(64, nmax // 2), nmax=nmax, nsteps=rng.randint(5, most),
                    every=rng.choice([0, 0, 5]), prec=prec)
    if kind == "forces":
        return dict(kind="forces", n=_log_int(rng, 8, 300000), prec=prec,
                    cloud=rng.choice(["gauss", "ellipsoid", "two_species", "two_species_grouped"]))
    if kind == "grad":
        return dict(kind="grad", n=_log_int(rng, 16, 100000), trap=rng.choice(["static", "rf"]), prec=prec,
                    cloud=rng.choice(["gauss", "two_species", "two_species_grouped", "crystal"]))
    if kind == "hvp":
        return dict(kind="hvp", n=_log_int(rng, 64, 32768), nvec=rng.randint(1, 8), trap="static", prec=prec,
                    cloud=rng.choice(["gauss", "two_species", "crystal"]))
    if kind == "autograd":
        return dict(kind="autograd", n=_log_int(rng, 16, 20000), cloud=rng.choice(["gauss", "two_species"]),
                    trap="static", prec=prec)
    steps = rng.randint(4, 24)
    return dict(kind="traj", n=_log_int(rng, 32, 8192), cloud=rng.choice(["gauss", "crystal"]), nsteps=steps,
                checkpoint=rng.randint(2, steps), prec=prec)


# ------------------------------------------------------------------- inputs
def _ions(case, seed):
    n, cloud = case["n"], case["cloud"]
    if cloud == "gauss":
        return inputs.cloud1024(n=n, seed=seed)
    if cloud == "ellipsoid":
        return inputs.rf32768(n=n, seed=seed)
    if cloud == "crystal":
        return inputs.crystal8192(n=n, seed=seed)
    d = inputs.cloud100k(n=n, seed=seed)
    return inputs.group_by_charge(d) if cloud == "two_species_grouped" else d


def _trap(case):
    if case["trap"] == "rf":
        return inputs.rf_trap(0.0, 0.3, 10.0e6, 0.1e6)
    trap = inputs.pseudo_trap(1.0e6, 1.0e6, 0.2e6)
    if case["trap"] == "damped":  # critical damping of the slowest axis, as the damped minimiser uses
        trap["gamma"] = 2.0 * trap["wz"] * inputs.MASS_40U
    return trap


def _sizes(case):
    """The runs' sizes: the same for every seed."""
    g = inputs.rng(inputs.BASE_SEED + 4)
    return g.integers(case["nmin"], case["nmax"] + 1, size=case["nrun"])


def _runs(case, seed):
    """The Kibble-Zurek recipe (``inputs.kz512``) at the case's sizes."""
    g, ns = inputs.rng(seed), _sizes(case)
    trap = inputs.ramp_trap(1.5e6, 0.6e6, 0.15e6, 0.0, 20e-6)
    pos, vel = [], []
    for n in ns:
        sigma = inputs.crystal_sigma(int(n), trap["wx"], trap["wy"], trap["wz"])
        pos.append(g.normal(size=(3, n)) * sigma[:, None])
        vel.append(inputs.maxwell(g, int(n), 10e-3, inputs.MASS_40U))
    pos, vel = np.concatenate(pos, axis=1), np.concatenate(vel, axis=1)
    n = pos.shape[1]
    return dict(x=pos[0], y=pos[1], z=pos[2], vx=vel[0], vy=vel[1], vz=vel[2], n=n, dt=2e-9,
                q=np.full(n, inputs.E_CHARGE), m=np.full(n, inputs.MASS_40U),
                offsets=np.concatenate([[0], np.cumsum(ns)]), traps=[dict(trap) for _ in ns])


def _vectors(n, nvec, seed):
    g = inputs.rng(seed + 7919)
    return g.normal(size=(nvec, 3, n))


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, kind=kind, prec=case["prec"])
    if kind in ("md", "ensemble"):
        d = _runs(case, seed) if kind == "ensemble" else _ions(case, seed)
        st = _dev(inputs.state9(d))
        s.update(state=[st[k] for k in range(9)], q=_dev(d["q"]), m=_dev(d["m"]), dt=d["dt"], t=0.0,
                 offsets=[int(o) for o in d["offsets"]] if kind == "ensemble" else None,
                 traps=d["traps"] if kind == "ensemble" else _trap(case))
        # the accelerations of the start, which the later calls carry on
        api.md_run(s["state"], s["q"], s["m"], s["traps"], 0.0, s["dt"], 0, offsets=s["offsets"], prec=s["prec"])
        return s
    d = _ions(case, seed)
    s.update(x=_dev(d["x"]), y=_dev(d["y"]), z=_dev(d["z"]), q=_dev(d["q"]), m=_dev(d["m"]))
    if kind in ("grad", "hvp", "autograd"):
        s["trap"] = _trap(case)
    if kind == "hvp":
        s["v"] = _dev(_vectors(case["n"], case["nvec"], seed))
    if kind == "autograd":
        s["r"] = torch.stack([s["x"], s["y"], s["z"]]).requires_grad_(True)
        s["v"] = _dev(_vectors(case["n"], 1, seed)[0])
    if kind == "traj":
        s["state0"] = _dev(inputs.state9(d))[:6].clone()
        s["trap"], s["dt"] = d["trap"], d["dt"]
    return s


def run(s):
    c, kind, prec = s["case"], s["kind"], s["prec"]
    if kind in ("md", "ensemble"):
        en = api.md_run(s["state"], s["q"], s["m"], s["traps"], s["t"], s["dt"], c["nsteps"], offsets=s["offsets"],
                        prec=prec, init_accel=False, every=c["every"])
        s["t"] += c["nsteps"] * s["dt"]
        return {"state": list(s["state"]), "energies": en}
    if kind == "forces":
        return list(api.coulomb_forces(s["x"], s["y"], s["z"], s["q"], prec=prec))
    if kind == "grad":
        g, u = api.coulomb_trap_grad(s["x"], s["y"], s["z"], s["q"], s["m"], s["trap"], 0.0, prec=prec, energy=True)
        return {"gradient": g, "energy": u}
    if kind == "hvp":
        return api.coulomb_hvp(s["x"], s["y"], s["z"], s["q"], s["v"], s["m"], s["trap"], prec=prec)
    if kind == "autograd":
        u = autograd.energy(s["r"], s["q"], s["m"], s["trap"], prec=prec)
        (g,) = torch.autograd.grad(u, s["r"], create_graph=True)
        (hv,) = torch.autograd.grad(g, s["r"], s["v"])
        return {"energy": u.detach(), "gradient": g.detach(), "product": hv}
    L, dldw, _ = drivers.traj_grad(s["state0"], s["q"], s["m"], s["trap"], s["dt"], c["nsteps"],
                                   checkpoint_every=c["checkpoint"], prec=prec)
    return {"msd": L, "gradient": dldw}


# Operations that the formulas cannot do without: an unordered pair's force
# (27: the pair's 20, the second ion's three accumulations and its charge), its
# energy (2), its Hessian product with B vectors (15 + 30 B).
_PAIR, _POT = 27.0, 2.0


def _hvp_pair(b):
    return 15.0 + 30.0 * b


def work(case):
    kind = case["kind"]
    if kind == "ensemble":
        ns = _sizes(case).astype(float)
        n1, pairs = float(ns.sum()), float(0.5 * (ns * (ns - 1.0)).sum())
        rec = case["nsteps"] // case["every"] + 1 if case["every"] else 0
        return {"bytes": 8.0 * n1 * (9 + 2 + 9), "flops": case["nsteps"] * _PAIR * pairs + rec * _POT * pairs}
    n = case["n"]
    pairs = 0.5 * n * (n - 1.0)
    if kind == "md":
        rec = case["nsteps"] // case["every"] + 1 if case["every"] else 0
        return {"bytes": 8.0 * n * (9 + 2 + 9), "flops": case["nsteps"] * _PAIR * pairs + rec * _POT * pairs}
    if kind == "forces":
        return {"bytes": 8.0 * n * 7, "flops": _PAIR * pairs}
    if kind == "grad":
        return {"bytes": 8.0 * n * 8, "flops": (_PAIR + _POT) * pairs}
    if kind == "hvp":
        return {"bytes": 8.0 * n * (5 + 6 * case["nvec"]), "flops": _hvp_pair(case["nvec"]) * pairs}
    if kind == "autograd":
        return {"bytes": 8.0 * n * (5 + 9), "flops": (_POT + 2 * _PAIR + _hvp_pair(1)) * pairs}
    # each step forward, recomputed forward, and one Hessian product back
    return {"bytes": 8.0 * n * 8 * case["nsteps"], "flops": case["nsteps"] * (2 * _PAIR + _hvp_pair(1)) * pairs}


# ------------------------------------------------------------------- exact
_KC = 1.0 / (4.0 * math.pi * 8.8541878128e-12)


def _blocks(n):
    step = max(1, min(n, (1 << 26) // n))
    return [(i, min(n, i + step)) for i in range(0, n, step)]


def _pairs(r, a, b):
    """Displacements (3, b - a, n) of the ions a .. b - 1 from all, and 1/r (0 for the ion itself)."""
    d = r[:, a:b, None] - r[:, None, :]
    y = torch.rsqrt((d * d).sum(0))
    y[torch.arange(b - a, device=r.device), torch.arange(a, b, device=r.device)] = 0.0
    return d, y


def _coulomb(r, q):
    """Forces (3, n) and energy, plain double loop in blocks."""
    F, U = torch.empty_like(r), r.new_zeros(())
    for a, b in _blocks(r.shape[1]):
        d, y = _pairs(r, a, b)
        w = q[None, :] * y
        U = U + 0.5 * (q[a:b] * w.sum(1)).sum()
        w = w * y * y
        F[:, a:b] = q[a:b] * (d * w).sum(2)
    return _KC * F, _KC * U


def _hessian(r, q, v):
    H = torch.empty_like(v)
    for a, b in _blocks(r.shape[1]):
        d, y = _pairs(r, a, b)
        w = q[None, :] * y ** 3
        for k in range(v.shape[0]):
            u = v[k][:, a:b, None] - v[k][:, None, :]
            H[k, :, a:b] = q[a:b] * ((3.0 * (d * u).sum(0) * y * y * d - u) * w).sum(2)
    return _KC * H


def _k(trap, t):
    wx, wy = trap["wx"], trap["wy"]
    if trap["kind"] == 1:
        w2 = trap["rf_omega"] ** 2
        kx = trap["rf_a"] * w2 / 4 + trap["rf_q"] * w2 / 2 * math.cos(trap["rf_omega"] * t + trap["rf_phase"])
        return kx, -kx, trap["wz"] ** 2
    if trap["t_ramp1"] > trap["t_ramp0"]:
        s = min(max((t - trap["t_ramp0"]) / (trap["t_ramp1"] - trap["t_ramp0"]), 0.0), 1.0)
        wx, wy = wx + s * (trap["wx1"] - wx), wy + s * (trap["wy1"] - wy)
    return wx * wx, wy * wy, trap["wz"] ** 2


def _col(k, like):
    return torch.tensor(k, dtype=like.dtype, device=like.device).reshape(3, 1)


def _md(st, q, m, trap, t0, dt, nsteps, every):
    """The run and its records, step by step."""
    r, v = st[:3].clone(), st[3:6].clone()
    F, U = _coulomb(r, q)
    a = F / m - _col(_k(trap, t0), r) * r
    recs, g = [], trap["gamma"] / m

    def record(t):
        K = 0.5 * (m * (v * v).sum(0)).sum()
        T = 0.5 * (m * (_col(_k(trap, t), r) * r * r).sum(0)).sum()
        recs.append(torch.stack([K, U, T, K + U + T]))

    if every:
        record(t0)
    for k in range(1, nsteps + 1):
        t = t0 + k * dt
        r = r + v * dt + 0.5 * dt * dt * (a - g * v)
        F, U = _coulomb(r, q)
        an = F / m - _col(_k(trap, t), r) * r
        v = (v * (1.0 - 0.5 * g * dt) + 0.5 * dt * (a + an)) / (1.0 + 0.5 * g * dt)
        a = an
        if every and k % every == 0:
            record(t)
    return torch.cat([r, v, a]), torch.stack(recs) if every else None


def exact(case, seed):
    kind = case["kind"]
    if kind == "ensemble":
        d = _runs(case, seed)
        st, q, m = _dev(inputs.state9(d)), _dev(d["q"]), _dev(d["m"])
        out, en = torch.empty_like(st), []
        for k in range(case["nrun"]):
            a, b = int(d["offsets"][k]), int(d["offsets"][k + 1])
            out[:, a:b], e = _md(st[:, a:b], q[a:b], m[a:b], d["traps"][k], 0.0, d["dt"], case["nsteps"],
                                 case["every"])
            en.append(e)
        return {"state": list(out), "energies": torch.stack(en) if case["every"] else None}
    d = _ions(case, seed)
    q, m, r = _dev(d["q"]), _dev(d["m"]), _dev(np.stack([d["x"], d["y"], d["z"]]))
    if kind == "md":
        st, en = _md(_dev(inputs.state9(d)), q, m, _trap(case), 0.0, d["dt"], case["nsteps"], case["every"])
        return {"state": list(st), "energies": en[None] if en is not None else None}
    if kind == "forces":
        return list(_coulomb(r, q)[0])
    if kind == "traj":
        return _traj(case, d, r, q, m)
    k = _col(_k(_trap(case), 0.0), r)
    if kind == "hvp":
        v = _dev(_vectors(case["n"], case["nvec"], seed))
        return _hessian(r, q, v) + m * k * v
    F, U = _coulomb(r, q)
    G, U = -F + m * k * r, U + 0.5 * (m * (k * r * r).sum(0)).sum()
    if kind == "grad":
        return {"gradient": G, "energy": U.reshape(1)}
    v = _dev(_vectors(case["n"], 1, seed))
    return {"energy": U, "gradient": G, "product": (_hessian(r, q, v) + m * k * v)[0]}


def _traj(case, d, r, q, m):
    """The discrete adjoint of the velocity-Verlet map, step by step."""
    n, dt, trap = case["n"], d["dt"], d["trap"]
    k, w = _col(_k(trap, 0.0), r), _col((trap["wx"], trap["wy"], trap["wz"]), r)
    accel = lambda r: _coulomb(r, q)[0] / m - k * r
    r0, v, a, path = r, _dev(np.stack([d["vx"], d["vy"], d["vz"]])), accel(r), []
    for _ in range(case["nsteps"]):
        r = r + v * dt + 0.5 * dt * dt * a
        an = accel(r)
        v, a = v + 0.5 * dt * (a + an), an
        path.append(r)
    L = float(((r - r0) ** 2).sum()) / n
    lr, lv, la = 2.0 * (r - r0) / n, torch.zeros_like(r), torch.zeros_like(r)
    grad = r.new_zeros(3)
    for r in reversed(path):
        s = la + 0.5 * dt * lv
        u = (s / m)[None]
        lr = lr - (_hessian(r, q, u) + m * k * u)[0]
        grad = grad + (-2.0 * w * r * s).sum(1)
        la = 0.5 * dt * lv + 0.5 * dt * dt * lr
        lv = lv + dt * lr
    return {"msd": L, "gradient": grad + (-2.0 * w * r0 * la).sum(1)}
