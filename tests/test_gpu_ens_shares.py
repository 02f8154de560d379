"""Ensembles of middle size take equal shares of all runs' pairs by default:
md_run against the persistent kernel (one workgroup per run, forced), for runs
that end at, just before and just after the edges of the units (16 j's), the
chunks (64 ions) and the blocks (256), every trap kind, records and none; and
the tiles of a large ensemble (forced), whose blocks' own pairs are taken by
Newton's third law, against the same."""
import numpy as np
import pytest

from paper_2106_11143_amd import inputs
from test_gpu_rows import M40, _cloud, api  # noqa: F401

pytestmark = pytest.mark.gpu
EDGES = [1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 271, 272, 273, 511, 512, 513, 1023, 4095, 4096]


def _run(api, sizes, prec, nsteps, every, init, cfg):
    from _gpu_util import dev
    parts = [_cloud(n, 900 + 3 * r) for r, n in enumerate(sizes)]
    st = np.concatenate([p[0] for p in parts], axis=1)
    q, m = (np.concatenate([p[k] for p in parts]) for k in (1, 2))
    base = parts[-1][3]
    kinds = [base, inputs.ramp_trap(1.5e6, 0.6e6, 0.15e6, 0.0, 20e-9), inputs.rf_trap(0.0, 0.3, 10e6, 0.15e6),
             dict(base, gamma=5e5 * M40)]
    traps = [kinds[r % 4] for r in range(len(sizes))]
    offs = np.concatenate([[0], np.cumsum(sizes)])
    if cfg:
        api.set_config("md_ensemble", offs[-1], prec, **cfg)
    try:
        ts = [dev(st[k]) for k in range(9)]
        en = api.md_run(ts, dev(q), dev(m), traps, 0.0, 1e-9, nsteps, offsets=offs, every=every, prec=prec,
                        init_accel=init)
        return np.stack([t.cpu().numpy() for t in ts]), en.cpu().numpy() if every else np.zeros((len(sizes), 1, 4))
    finally:
        api.reset_config("md_ensemble", offs[-1], prec)


def _agree(a, b, sizes):
    """The same sums in another order: as the other tests of the paths."""
    offs = np.concatenate([[0], np.cumsum(sizes)])
    for blk in (slice(0, 3), slice(3, 6), slice(6, 9)):
        assert np.abs(a[0][blk] - b[0][blk]).max() <= 1e-11 * np.abs(b[0][blk]).max(), blk
    for r, n in enumerate(sizes):  # run by run: a small run's error does not hide behind a large one's size
        x, y = a[0][:3, offs[r]:offs[r + 1]], b[0][:3, offs[r]:offs[r + 1]]
        assert np.abs(x - y).max() <= 1e-11 * np.abs(y).max(), (r, n)
        assert np.abs(a[1][r] - b[1][r]).max() <= 1e-11 * max(np.abs(b[1][r]).max(), 1e-300), (r, n)


PERSISTENT = dict(p=4, wg=512, splits=1, algo=0)


@pytest.mark.parametrize("sizes", [EDGES + [3000] * 10, [4096, 4081] * 5 + EDGES[::-1], [2048] * 40])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_shares(api, sizes, prec):  # noqa: F811
    for nsteps, every, init in ((0, 1, True), (5, 2, True), (4, 0, False)):
        _agree(_run(api, sizes, prec, nsteps, every, init, None),
               _run(api, sizes, prec, nsteps, every, init, PERSISTENT), sizes)
    assert api.poll_flags() == 0


@pytest.mark.parametrize("prec", ["fp64", "ieee"])
def test_tiles_of_a_large_ensemble(api, prec):  # noqa: F811
    sizes = [4096] * 34 + EDGES
    want = _run(api, sizes, prec, 2, 2, True, PERSISTENT)
    for jl in (256, 512):
        _agree(_run(api, sizes, prec, 2, 2, True, dict(p=4, wg=4, splits=jl, algo=2)), want, sizes)
    assert api.poll_flags() == 0


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_two_wave_finish(api, prec):  # noqa: F811
    """From 4096 chunks of 64 ions on, two waves finish a chunk instead of
    eight."""
    g = np.random.Generator(np.random.PCG64(17))
    sizes = [n for n in EDGES if n <= 1024] + [int(n) for n in g.integers(64, 1025, 560)]
    units = pairs = 0
    for n in sizes:  # the rule that picks the path: rows, shares and tiles by estimated time
        nI, C = -(-n // 256), -(-n // 16)
        units += nI * C - 16 * (nI * (nI - 1) // 2)
        pairs += n * n
    assert sum(-(-n // 64) for n in sizes) >= 4096
    assert 15e-6 + 3.3e-9 * units < min(5e-6 + pairs / 1.25e12, 40e-6 + 3e-9 * units)
    for nsteps, every, init in ((0, 1, True), (4, 2, True), (3, 0, False)):
        _agree(_run(api, sizes, prec, nsteps, every, init, None),
               _run(api, sizes, prec, nsteps, every, init, PERSISTENT), sizes)
    assert api.poll_flags() == 0
