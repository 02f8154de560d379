"""Tuned entries at the sizes of their bucket that take another path: the calls
run, in the workspace that cb_workspace_size gives them, and return bitwise what
untuned calls return."""
import json

import numpy as np
import pytest

from test_gpu_rows import _cloud, api  # noqa: F401

pytestmark = pytest.mark.gpu
OPS = ("forces", "energy", "md_step", "md_run")


def _results(api, n):
    import torch
    from _gpu_util import dev, state_tensors
    api.clear_workspace_cache()
    st, q, m, trap = _cloud(n, n)
    x, y, z, q, m = *(dev(c) for c in st[:3]), dev(q), dev(m)
    g, u = api.coulomb_trap_grad(x, y, z, q, m, trap, energy=True)
    ts = state_tensors(st)
    en = api.md_run(ts, q, m, trap, 0.0, 1e-9, 2, every=2)
    return [*api.coulomb_forces(x, y, z, q), api.coulomb_energy(x, y, z, q), g, u, torch.stack(ts), en]


def _drop(api, *ns):
    for op in OPS:
        for n in ns:
            api.reset_config(op, n)


@pytest.mark.parametrize("tuned,n", [(5000, 7000), (7000, 5000), (39900, 33500), (300001, 262145)])
def test_another_path_in_the_bucket(api, tmp_path, tuned, n):  # noqa: F811
    import torch
    want = _results(api, n)
    f = tmp_path / "tune.jsonl"
    base = dict(arch=torch.cuda.get_device_properties(0).gcnArchName.split(":")[0])
    f.write_text("\n".join(json.dumps(dict(base, op=op, prec=0, bucket=0, n=tuned, p=1, wg=64, splits=8, algo=0))
                           for op in range(4) if api.get_path(op, n) != "config") + "\n")
    api.load_tuning(str(f))
    try:
        for op in OPS:
            assert api.get_config(op, n)["tuned"] == (api.get_path(op, n) != "config")
        for a, b in zip(_results(api, n), want):
            assert torch.equal(a, b)
    finally:
        _drop(api, n, tuned)


def test_tuning_times_the_bands(api):  # noqa: F811
    """Beyond 2^18 ions the bands take two thirds of the direct kernel's time:
    the tuned calls take them."""
    n = 262145
    try:
        api.autotune("energy", n)
        assert api.get_config("energy", n)["tuned"] and api.get_path("energy", n) == "bands"
    finally:
        _drop(api, n)


@pytest.mark.parametrize("op,n", [("md_run", 300), ("md_step", 5000), ("forces", 7000), ("md_run", 8192), ("md_run", 9000)])
def test_file_restores_what_tuning_set(api, tmp_path, op, n):  # noqa: F811
    f = str(tmp_path / "tune.jsonl")
    entries = lambda: {(o, k): (api.get_config(o, k), api.get_path(o, k)) for o in OPS for k in (n, 3 * n // 4)}  # noqa: E731
    untuned = entries()
    try:
        api.autotune(op, n, "fp64", f)
        tuned = entries()
        assert tuned["forces", n][0]["tuned"]
        _drop(api, n)
        assert entries() == untuned
        api.load_tuning(f)
        assert entries() == tuned
    finally:
        _drop(api, n)
