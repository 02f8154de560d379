"""cb_rows_run_spins validates its arguments before it touches a device, as
md_run does."""
import ctypes as C

from test_abi_cpu import _ws, api  # noqa: F401


def test_argument_errors(api):  # noqa: F811
    L = api.lib()
    a = [C.c_void_p((k + 1) << 24) for k in range(11)]
    good = dict(n=500, s=api.State(*a[:9]), q=a[9], m=a[10], trap=api.make_trap(dict(kind=0, wx=1e6, wy=1e6, wz=1e5)),
                t0=0.0, dt=1e-9, nsteps=20, eps2=0.0, prec=0, energies=C.c_void_p(12 << 24), every=1, spins=0, ws=_ws(),
                ws_bytes=1 << 40)
    ref = lambda v: C.byref(v) if isinstance(v, C.Structure) else v  # noqa: E731

    def call(**kw):
        return L.cb_rows_run_spins(*[ref(v) for v in dict(good, **kw).values()], None), api.last_error()

    inside = C.c_void_p((1 << 24) + 8)
    for kw, word in ((dict(s=None), "NULL"), (dict(q=None), "NULL"), (dict(m=None), "NULL"), (dict(trap=None), "NULL"),
                     (dict(s=api.State(*a[:8], None)), "NULL"), (dict(ws=None), "NULL"),
                     (dict(ws=C.c_void_p(8)), "aligned"), (dict(s=api.State(*a[:8], a[0])), "overlap"),
                     (dict(q=inside), "overlap"), (dict(every=0), "every"), (dict(dt=0.0), "dt"),
                     (dict(t0=float("nan")), "t0"), (dict(eps2=-1.0), "eps2"), (dict(prec=9), "precision"),
                     (dict(n=0), "n = 0"), (dict(trap=api.make_trap(dict(kind=3))), "kind"),
                     (dict(nsteps=2), "not a run"), (dict(n=2000), "not a run"), (dict(ws_bytes=100), "not a run")):
        status, msg = call(**kw)
        assert status == api.CB_EINVAL and word in msg, (kw, msg)
    assert call(prec=4)[0] == api.CB_EUNSUPPORTED
