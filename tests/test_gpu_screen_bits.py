"""Screened against unscreened, bit for bit: the same spectra searched with a
screening pass, without one (a tile budget that leaves its records no room)
and through the no-alloc workspace must give the same powers and the same
cells, in every arithmetic, with the kernels compiled for the lattice and the
static ones.  That the first search is screened and the second is not is
asserted on the CPU for the same shapes (test_host_routes.py).

The unscreened kernels against the FP64 oracle: the one-wave form (4096
segments or more, no screening on n_mbd = 64 and 128) and the work-group form
on the same data."""
import numpy as np
import pytest
import torch

from oracle import frb_oracle as O
from paper_1801_02391_amd import frbx

from gpu_helpers import compare_powers, note, oracle_cube
from screen_shapes import K, LATTICES, N_DM, SCREENED, WINDOWS

pytestmark = pytest.mark.gpu


POWER_TOL = 4e-6   # separate compilations of the same float32 sums


def _params(name, J, P, R, precision, n_dm=N_DM, n_mbd=256):
    f0 = LATTICES[name]
    lay = dict(n_baselines=1, if_freq_mhz=f0, n_if=len(f0), n_chan=J, chan_bw_mhz=32.0 / J, t_ap_ms=1.0, n_frames=K)
    return lay, dict(dm_lo=0.0, dm_step=0.0, n_dm=n_dm, sbd_pad=P, n_mbd=n_mbd, n_rate=R, windows=WINDOWS, threshold=3.0,
                     n_win_min=1, n_bl_min=1, precision=precision)


def _search(V, *shape, budget=0, specialise=True, **kw):
    lay, par = _params(*shape, **kw)
    s = frbx.Search(lay)
    s.configure(par)
    s.set_specialisation(specialise)
    if budget:
        s.set_tile_budget(budget)
    s.load(torch.from_numpy(V).to("cuda:0"))
    s.run()
    return s, *s.power_cube()


def _noise(name, J, seed):
    """Noise, a channel far above it in the second half of the record."""
    g = np.random.default_rng(seed)
    V = (g.standard_normal((1, len(LATTICES[name]), J, K)) + 1j * g.standard_normal((1, len(LATTICES[name]), J, K)))
    V[:, 0, J // 2 + 1, K // 2:] *= 200.0
    return V.astype(np.complex64)


@pytest.mark.parametrize("specialise", [True, False])
@pytest.mark.parametrize("name,J,P,R,precision", SCREENED)
def test_screened_search_keeps_every_bit(name, J, P, R, precision, specialise):
    if precision != "f32" and not specialise:
        pytest.skip("only the float32 kernels are compiled for a lattice")
    note(f"screen bits {name} J={J} P={P} R={R} {precision} specialise={specialise}")
    V = _noise(name, J, 5)
    s, p, i = _search(V, name, J, P, R, precision, specialise=specialise)
    _, p0, i0 = _search(V, name, J, P, R, precision, budget=8 * len(LATTICES[name]) * J * K, specialise=specialise)
    assert np.array_equal(p.view(np.uint32), p0.view(np.uint32)) and np.array_equal(i, i0)
    pn = torch.empty(p.size, device="cuda:0")
    idx = torch.empty(p.size, dtype=torch.int32, device="cuda:0")
    assert s.run_cube_noalloc(pn, idx) == p.size
    torch.cuda.synchronize()
    assert np.array_equal(pn.cpu().numpy(), p.ravel()) and np.array_equal(idx.cpu().numpy(), i.ravel())


@pytest.mark.parametrize("name,J,M,P,R", [("1if", 8, 16, 4, 1), ("5if-compact", 16, 64, 2, 3), ("3if-spread", 32, 128, 4, 3),
                                          ("16if-compact", 32, 128, 1, 2), ("8if-compact", 64, 64, 8, 2),
                                          ("3if-spread", 64, 128, 4, 9), ("5if-compact", 16, 256, 1, 2)])
def test_one_wave_per_segment_against_the_oracle_and_the_work_group_form(name, J, M, P, R):
    note(f"wave form {name} J={J} M={M} P={P} R={R}")
    V = _noise(name, J, 9)
    shape = (name, J, P, R, "f32")
    _, p, i = _search(V, *shape, n_mbd=M)
    _, p0, i0 = _search(V, *shape, n_dm=1, n_mbd=M)
    assert p.size >= 4096 > p0.size   # one wave and one work-group per segment
    assert np.all(np.abs(p[:, :1] - p0) <= POWER_TOL * p0)
    lay, par = _params(*shape, n_dm=1, n_mbd=M)
    res = O.search(V, lay, par)
    po, io, s2 = oracle_cube(res, 1, 1, res["grids"]["segs"])
    for got_p, got_i in ((p[:, :1], i[:, :1]), (p[:, -1:], i[:, -1:]), (p0, i0)):
        compare_powers(got_p, got_i, po, io, s2, name)
