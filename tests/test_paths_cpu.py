"""cb_get_path: the path that a call takes in the place of the launches that
cb_get_config reports, at both sides of every line between them, and that it
follows forced entries."""
import pytest

from test_abi_cpu import api  # noqa: F401

FORCE_OPS = ("forces", "energy", "md_step", "md_run")


@pytest.mark.parametrize("n,path", [
    (1, "rows"), (6144, "rows"), (6145, "shares"), (32767, "shares"), (32768, "config"), (33500, "shares"),
    (39900, "config"), (57344, "shares"), (57345, "config"), (262144, "config"), (262145, "bands"),
    (1 << 28, "bands")])
def test_untuned(api, n, path):  # noqa: F811
    for op in FORCE_OPS:
        for prec in ("fp64", "mixed", "ieee", "fp32"):
            api.reset_config(op, n, prec)  # (an entry that another test left)
            assert api.get_path(op, n, prec) == path
    assert api.get_path("forces", n, "mixed_f32d") == "config"
    assert api.get_path("hvp", n) == api.get_path("adjoint", n) == "config"


def test_forced_entries_run_as_set(api):  # noqa: F811
    for n, cfg in ((5000, dict(p=1, wg=64, splits=8, algo=0)), (12000, dict(p=4, wg=4, splits=256, algo=2)),
                   (300000, dict(p=1, wg=64, splits=64, algo=0))):
        for op in FORCE_OPS:
            api.reset_config(op, n, "fp64")
            api.reset_config(op, n, "mixed")
            untuned = api.get_path(op, n)
            assert untuned != "config"
            api.set_config(op, n, "fp64", **cfg)
            try:
                assert api.get_path(op, n) == "config"
                assert api.get_path(op, n, "mixed") == untuned
            finally:
                api.reset_config(op, n)
            assert api.get_path(op, n) == untuned


def test_bad_arguments(api):  # noqa: F811
    L = api.lib()
    import ctypes as C
    out = C.c_int32(-1)
    assert L.cb_get_path(0, 100, 0, None) == api.CB_EINVAL
    for op, n, prec in ((-1, 100, 0), (6, 100, 0), (7, 100, 0), (0, 0, 0), (0, (1 << 28) + 1, 0), (0, 100, 5), (0, 100, -1)):
        assert L.cb_get_path(op, n, prec, C.byref(out)) == api.CB_EINVAL
    assert out.value == -1
