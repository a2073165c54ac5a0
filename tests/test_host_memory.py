"""Device memory of a search, on the CPU: the library's host code against a
stand-in device (fake_device.cpp: quota, refused allocations, launches named
instead of run)."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIBDIR = os.path.join(os.path.dirname(HERE), "paper_1801_02391_amd")
NOMEM = 4

# 3 IFs x 16 channels, 64 rates: records of 13 times the spectra
MANY_RATES = dict(J=16, P=8, R=64, K=20000, D=40, W="1,2,4,8", **{"if": "3000,3032,5240"})
BASELINES = dict(J=32, P=4, R=8, K=2000, B=6, D=3, W="2,4", **{"if": "3000,3032,5240"})


@pytest.fixture(scope="module")
def device(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fake") / "fake_device")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-rdynamic", os.path.join(HERE, "fake_device.cpp"),
                    "-L", LIBDIR, "-lfrbx", f"-Wl,-rpath,{LIBDIR}", "-o", exe], check=True)

    def run(**arg):
        r = subprocess.run([exe, *(f"{k}={v}" for k, v in arg.items())], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
        out = r.stdout
        get = lambda k: int(m.group(1)) if (m := re.search(rf"^{k} (\d+)", out, re.M)) else None
        return dict(text=out, status=get("status"), peak=get("peak"), segments=get("segments"),
                    screened=out.count("screen_kernel"), refused=out.count("refused"))

    return run


def results(shape, segments):
    """Bytes of a run's cube and crossing list, and room for its statistics."""
    cube = shape.get("B", 1) * shape["D"] * segments
    return 8 * cube + 48 * max(1 << 16, cube // 64) + (1 << 20)


def spectra(shape):
    return 8 * len(shape["if"].split(",")) * shape["J"] * shape["K"]


@pytest.mark.parametrize("shape", [MANY_RATES, BASELINES])
@pytest.mark.parametrize("trials,screened", [(1.0, False), (1.5, False), (20.0, True)])
def test_tiles_and_records_stay_within_the_budget(device, shape, trials, screened):
    budget = int(trials * spectra(shape))
    r = device(**shape, budget=budget)
    assert r["status"] == 0 and r["refused"] == 0
    assert r["peak"] <= budget + results(shape, r["segments"])
    if shape is MANY_RATES:
        assert (r["screened"] > 0) == screened


def test_a_budget_below_one_trial_is_refused(device):
    assert device(**MANY_RATES, budget=spectra(MANY_RATES) - 1)["status"] == NOMEM


@pytest.mark.parametrize("shape", [MANY_RATES, BASELINES])
def test_a_search_that_fits_without_records_runs(device, shape):
    """Quotas from the spectra and the results alone up to what a run takes."""
    most = device(**shape)
    least = device(**shape, quota=1)
    assert least["status"] == NOMEM
    need = shape["D"] * spectra(shape) + results(shape, most["segments"])
    assert need < most["peak"]
    for k in range(9):
        r = device(**shape, quota=need + (most["peak"] - need) * k // 8)
        assert r["status"] == 0, (k, r["text"][-300:])
    assert r["screened"] == most["screened"] > 0


@pytest.mark.parametrize("shape", [MANY_RATES, BASELINES])
def test_one_refused_allocation_is_enough_only_for_what_a_run_needs(device, shape):
    """Every allocation of a first run refused once: the records' refusal only
    costs the screening; any other is an error, unless the tile holds several
    baselines and the run is tried again with one."""
    tolerated = 0
    for k in range(1, 12):
        r = device(**shape, refuse=k)
        if not r["refused"]:
            break
        assert r["status"] in (0, NOMEM)
        tolerated += r["status"] == 0
    assert k > 7 and tolerated == (k - 1 if shape is BASELINES else 1)


def test_records_are_given_back_for_a_chunked_search(device):
    """Pushes whose later, larger passes need the memory that the records of
    an earlier one hold."""
    shape = dict(MANY_RATES, D=8, mode="stream", chunk=4000, pushes=3)
    most = device(**shape)
    assert most["status"] == 0 and most["screened"] > 0
    for k in range(4, 9):
        r = device(**shape, quota=most["peak"] * k // 8)
        assert r["status"] == 0, (k, r["text"][-300:])
