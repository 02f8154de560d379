"""cb_get_path: the path that a call takes in the place of the launches that
cb_get_config reports, at both sides of every line between them, and that it
follows forced entries."""
import pytest

from test_abi_cpu import api  # noqa: F401

FORCE_OPS = ("forces", "energy", "md_step", "md_run")


@pytest.mark.parametrize("n,path", [
    (1, "rows"), (2400, "rows"), (2401, "rows"), (6144, "rows"), (6145, "shares"), (8750, "shares"), (8751, "shares"), (32767, "shares"), (32768, "config"), (33500, "shares"),
    (39900, "config"), (57344, "shares"), (57345, "config"), (262144, "config"), (262145, "bands"),
    (1 << 28, "bands")])
def test_untuned(api, n, path):  # noqa: F811
    for op in FORCE_OPS:
        for prec in ("fp64", "mixed", "ieee", "fp32"):
            api.reset_config(op, n, prec)  # (an entry that another test left)
            if op == "energy" and 2400 < n <= (8750 if prec in ("mixed", "fp32") else 6144):
                assert api.get_path(op, n, prec) == "config"  # the potential alone
            else:
                assert api.get_path(op, n, prec) == path
            if op == "energy":  # the gradient with the energy
                assert api.get_path("grad", n, prec) == path
    assert api.get_path("forces", n, "mixed_f32d") == "config"
    assert api.get_path("hvp", n) == api.get_path("adjoint", n) == "config"


def test_forced_entries_run_as_set(api):  # noqa: F811
    for n, cfg in ((5000, dict(p=1, wg=64, splits=8, algo=0)), (12000, dict(p=4, wg=4, splits=256, algo=2)),
                   (300000, dict(p=1, wg=64, splits=64, algo=0))):
        for op in FORCE_OPS:
            api.reset_config(op, n, "fp64")
            api.reset_config(op, n, "mixed")
            untuned = api.get_path(op, n)
            assert untuned != "config" or op == "energy"
            api.set_config(op, n, "fp64", **cfg)
            try:
                assert api.get_path(op, n) == "config"
                assert api.get_path(op, n, "mixed") == untuned
            finally:
                api.reset_config(op, n)
            assert api.get_path(op, n) == untuned


def test_gradient_with_the_energy(api):  # noqa: F811
    """Its configuration is the energy's: a forced one runs as set; its workspace
    holds the shares that it takes where neither energy nor forces take them."""
    for n, untuned in ((5000, "rows"), (7000, "shares")):
        api.reset_config("energy", n)
        assert api.get_path("grad", n) == untuned
        api.set_config("energy", n, "fp64", p=1, wg=64, splits=8, algo=0)
        assert api.get_path("grad", n) == "config"
        api.reset_config("energy", n)
    n = 7000
    api.reset_config("forces", n, "fp32")
    size = api.workspace_size("grad", n, prec="fp32")
    assert (api.get_path("energy", n, "fp32"), api.get_path("grad", n, "fp32")) == ("config", "shares")
    api.set_config("forces", n, "fp32", p=1, wg=64, splits=8, algo=0)
    try:
        assert api.workspace_size("grad", n, prec="fp32") == size
    finally:
        api.reset_config("forces", n, "fp32")


def test_bad_arguments(api):  # noqa: F811
    L = api.lib()
    import ctypes as C
    out = C.c_int32(-1)
    assert L.cb_get_path(0, 100, 0, None) == api.CB_EINVAL
    for op, n, prec in ((-1, 100, 0), (6, 100, 0), (8, 100, 0), (0, 0, 0), (0, (1 << 28) + 1, 0), (0, 100, 5), (0, 100, -1)):
        assert L.cb_get_path(op, n, prec, C.byref(out)) == api.CB_EINVAL
    assert out.value == -1


OP = {"forces": 0, "energy": 1, "md_step": 2, "md_run": 3, "hvp": 4}
PATH = {"config": 0, "rows": 1, "shares": 2, "bands": 3}


def _load(api, tmp_path, *lines):
    """A tuning file of these (op, n, algo, path, base) lines: path and base
    None where the file was written without them."""
    f = tmp_path / "tune.jsonl"
    out = []
    for op, n, algo, path, base in lines:
        shape = {0: (1, 64, 8), 2: (4, 4, 256), 3: (1, 64, 4), 4: (8, 4, 512)}[algo]
        t = '"op": %d, "prec": 0, "bucket": 0, "n": %d, "p": %d, "wg": %d, "splits": %d, "algo": %d' % (
            OP[op], n, *shape, algo)
        t += "" if path is None else ', "path": %d' % PATH[path]
        t += "" if base is None else ', "base": %d' % PATH[base]
        # (an architecture that is not this machine's: the line is skipped)
        out += ['{"arch": "%s", %s, "ms": 1.0}' % (arch, t) for arch in ("unknown", "gfx950")]
    f.write_text("\n".join(out) + "\n")
    api.load_tuning(str(f))


@pytest.fixture
def clean(api):  # noqa: F811
    def drop():
        for op in FORCE_OPS:
            for b in range(12, 20):
                api.reset_config(op, 1 << b)
    drop()
    yield
    drop()


# (line, {n: path}): the line's path at the sizes of its bucket that have the
# default it was timed against, their default at the others; a line that does
# not say what it was timed against takes the default everywhere, except that
# rows and shares were always timed when a path was written at all.
@pytest.mark.parametrize("line,want", [
    (("forces", 300001, 0, None, None), {262145: "bands", 300001: "bands"}),
    (("forces", 300001, 0, "config", None), {262145: "bands", 300001: "bands"}),
    (("forces", 300001, 0, "config", "bands"), {262145: "config", 300001: "config"}),
    (("energy", 300001, 0, "bands", "bands"), {262145: "bands"}),
    (("md_run", 300001, 0, "bands", "bands"), {262145: "bands"}),
    (("forces", 65536, 2, "config", "config"), {33500: "shares", 39900: "config", 57344: "shares", 60000: "config"}),
    (("md_step", 39900, 2, "config", "config"), {33500: "shares", 39900: "config", 57344: "shares", 65536: "config"}),
    (("energy", 12000, 2, "config", None), {9000: "config", 12000: "config"}),
    (("energy", 12000, 2, "shares", "shares"), {9000: "shares", 16384: "shares"}),
    (("energy", 12000, 2, None, None), {9000: "shares", 12000: "shares"}),
    (("forces", 7000, 0, "config", "shares"), {5000: "rows", 7000: "config"}),
    (("forces", 5000, 0, "config", "rows"), {5000: "config", 7000: "shares"}),
    (("forces", 5000, 0, "shares", "rows"), {5000: "shares", 7000: "shares"}),
    (("forces", 5000, 0, "bands", "rows"), {5000: "rows"}),
    (("md_run", 5000, 3, "rows", "rows"), {5000: "rows", 7000: "shares"}),
    (("md_run", 7000, 3, "rows", "shares"), {5000: "rows", 7000: "rows"}),
    (("md_run", 7000, 3, "config", None), {5000: "rows", 7000: "rows"})])
def test_tuned_at_one_size(api, clean, tmp_path, line, want):  # noqa: F811
    _load(api, tmp_path, line)
    op = line[0]
    for n, path in want.items():
        assert api.get_config(op, n)["tuned"]
        assert api.get_path(op, n) == path, n
    if op.startswith("md") or line[1] > 8192 and op == "forces":
        for n, path in want.items():
            assert api.get_path("md_step", n) == api.get_path("md_run", n) == path


# What tuning forces and an md call at up to 8192 ions had set comes back from
# its file: the forces' entry is not the md calls'.  As written now (a forces
# line and an md line), and as two md lines by files without "base".
@pytest.mark.parametrize("lines,forces,md", [
    ([("forces", 5000, 0, "rows", "rows"), ("md_run", 5000, 0, "shares", "rows")], (0, "rows"), (0, "shares")),
    ([("forces", 5000, 2, "config", "rows"), ("md_run", 5000, 3, "rows", "rows")], (2, "config"), (3, "rows")),
    ([("md_run", 5000, 3, "rows", "rows")], None, (3, "rows")),
    ([("md_run", 5000, 0, "config", "rows")], None, (0, "config")),
    ([("forces", 5000, 2, "config", "rows")], (2, "config"), None),
    ([("md_step", 5000, 2, "rows", None), ("md_run", 5000, 0, "config", None)], (2, "rows"), (0, "config")),
    ([("md_run", 5000, 2, "rows", None), ("md_run", 5000, 0, "shares", None)], (2, "rows"), (0, "shares")),
    ([("md_run", 5000, 2, "rows", None), ("md_run", 5000, 3, "config", None)], (2, "rows"), (3, "rows")),
    ([("md_run", 5000, 2, "rows", None), ("md_run", 5000, 0, "shares", None),
      ("md_run", 5000, 0, "config", None), ("md_run", 5000, 0, "rows", None)], (0, "config"), (0, "rows")),
    ([("md_run", 5000, 2, None, None), ("md_run", 5000, 0, None, None)], (2, "rows"), (0, "rows"))])
def test_files_of_small_runs(api, clean, tmp_path, lines, forces, md):  # noqa: F811
    _load(api, tmp_path, *lines)
    for op, want in (("forces", forces), ("md_step", md), ("md_run", md)):
        c = api.get_config(op, 5000)
        assert c["tuned"] == (want is not None), op
        if want:
            assert (c["algo"], api.get_path(op, 5000)) == want, op
