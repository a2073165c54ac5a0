"""Which kernels a search takes, on the CPU: the library's host code against a
stand-in device that names the launches (fake_device.cpp)."""
import re

import pytest

from screen_shapes import K, LATTICES, N_DM, PRECISION, SCREENED, WHOLE, WINDOWS
from test_host_memory import MANY_RATES, device, spectra  # noqa: F401  (a fixture)


def kernels(text):
    """The search kernels of a run: screening pass, find_kernel, and the form's
    own kernel as (channels, evaluates candidates, threads per segment)."""
    out = set()
    for name in re.findall(r"^kernel (.*) grid", text, re.M):
        if m := re.search(r"(screen|find)_kernel", name):
            out.add(m.group(1))
        elif m := re.search(r"fringe_kernel(?:ILi|<)(\d+)(?:ELi|, )\d+(?:ELb|, )\w+(?:ELb|, )\w+(?:ELb|, )\w+(?:ELj|, )"
                            r"\d+u?(?:ELb|, )(\w+)(?:ELi|, )(\d+)", name):
            out.add((int(m.group(1)), m.group(2) in ("1", "true"), int(m.group(3))))
        elif m := re.search(r"fringe_mfma_kernelILi(\d+)ELi\dELi\dELb0ELb(\d)E", name):
            out.add((int(m.group(1)), m.group(2) == "1", 256))
    return out


def form(precision):
    return dict(prec=PRECISION[precision])


@pytest.mark.parametrize("jit", [0, 1])
@pytest.mark.parametrize("precision", ["f32", "f16x3"])
def test_without_records_every_cell_by_the_plain_kernel(device, precision, jit):  # noqa: F811
    """The records do not fit the budget, the device refuses them, or they do
    not fit beside the spectra in the no-alloc workspace (which compiles
    nothing)."""
    shape = dict(MANY_RATES, jit=jit, **form(precision))
    wave = 64 if precision == "f32" else 256
    r = device(**shape, budget=spectra(shape))
    assert r["status"] == 0 and kernels(r["text"]) == {(16, False, wave)}
    r = device(**shape)
    assert r["status"] == 0 and "screen" in kernels(r["text"])
    n = next(k for k in range(1, 12) if device(**shape, refuse=k)["status"] == 0)
    r = device(**shape, refuse=n)
    first = r["text"].split("mark again")[0]
    assert r["refused"] == 1 and kernels(first) == {(16, False, wave)}
    r = device(**shape, mode="noalloc")
    assert r["status"] == 0 and kernels(r["text"]) == {(16, False, wave)}
    assert "compiled" not in r["text"].split("prepared")[1]
    assert ("jit:" in r["text"]) == (jit == 1 and precision == "f32")


def test_a_screened_search_compiles_the_plain_kernel_only_where_it_may_need_it(device):  # noqa: F811
    vgos = dict(J=64, P=4, R=8, W="2,4,8", **{"if": ",".join(map(str, LATTICES["32if-vgos"]))})
    for arg in (dict(K=400, D=4), dict(K=400, D=4, mode="noalloc"), dict(K=6000, D=2)):
        r = device(**vgos, **arg)
        assert kernels(r["text"]) == {"screen", "find", (64, True, 256)}
        assert re.findall(r"^compiled frbx::(\w+)<", r["text"], re.M) == ["fringe_kernel", "find_kernel"]


def shape(name, J, P, R, precision, **kw):
    return dict(J=J, P=P, R=R, W=",".join(map(str, WINDOWS)), **form(precision), **{"if": ",".join(map(str, LATTICES[name]))}, **kw)


@pytest.mark.parametrize("case", SCREENED)
def test_searches_that_are_screened(device, case):  # noqa: F811
    s = shape(*case, K=K, D=N_DM)
    own = {k for k in kernels(device(**s)["text"]) if isinstance(k, tuple)}
    assert own == {(case[1], True, 256)} and "screen" in kernels(device(**s)["text"])
    assert "screen" not in kernels(device(**s, budget=spectra(s))["text"])   # no room for the records


@pytest.mark.parametrize("case", WHOLE)
def test_searches_that_are_evaluated_whole(device, case):  # noqa: F811
    k, = kernels(device(**shape(*case, K=K, D=N_DM))["text"])
    assert k[:2] == (case[1], False)


# (lattice, channels, sbd_pad, rates, precision), MBD points, DM trials, APs a push: kernels
PUSHES = [
    (("32if-vgos", 64, 4, 1, "f32"), 256, 2, 64, {(64, False, 256)}),
    (("32if-vgos", 64, 4, 1, "f32"), 256, 8, 4096, {"screen", "find", (64, True, 256)}),
    (("32if-vgos", 64, 4, 8, "f32"), 256, 2, 16, {"screen", "find", (64, True, 256)}),
    (("8if-compact", 32, 4, 1, "f32"), 256, 8, 16, {(32, False, 256)}),
    (("8if-compact", 32, 4, 1, "f32"), 256, 8, 4096, {"screen", "find", (32, True, 256)}),
    (("8if-compact", 64, 8, 8, "f32"), 128, 2, 64, {(64, False, 256)}),
    (("8if-compact", 64, 8, 8, "f32"), 128, 4, 4096, {(64, False, 64)}),
    (("32if-vgos", 64, 4, 1, "f16x3"), 256, 2, 64, {(64, False, 256)}),
    (("32if-vgos", 64, 4, 8, "f16x3"), 256, 2, 16, {"screen", (64, True, 256)}),
    (("32if-vgos", 64, 4, 8, "f16"), 256, 2, 16, {"screen", (64, True, 256)}),
    (("32if-vgos", 64, 4, 4, "f16"), 256, 2, 64, {(64, False, 256)}),
]


@pytest.mark.parametrize("frames", [50, 20000])
@pytest.mark.parametrize("case,M,D,chunk,want", PUSHES)
def test_a_push_takes_the_kernels_of_its_own_size(device, case, M, D, chunk, want, frames):  # noqa: F811
    """Whatever the number of frames of the layout."""
    r = device(**shape(*case, M=M, D=D, K=frames), mode="stream", chunk=chunk)
    assert r["status"] == 0 and kernels(r["text"].split("mark push 1")[1]) == want


@pytest.mark.parametrize("refuse", [0, 1, 2, 3])
def test_a_run_after_a_stream_of_another_size(device, refuse):  # noqa: F811
    """A run too small to be screened, after a stream whose pushes are: also
    where the stream's tables or buffers were refused."""
    case = ("32if-vgos", 64, 4, 1, "f32")
    r = device(**shape(*case, K=50, D=8), mode="mixed", chunk=4096, refuse=refuse)
    began, ran = re.split("mark run", r["text"].split("mark stream ")[1])
    assert r["status"] == 0 and began[0] == ("4" if refuse else "0")
    assert kernels(began) in ({(64, False, 256)}, {"screen", "find", (64, True, 256)})
    assert kernels(ran) == {(64, False, 256)}
