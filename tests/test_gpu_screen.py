"""The screened search (float16 screening pass, then the candidate units in
the form's own arithmetic) against every cell of its segments, as
frbx_dump_segment evaluates them without a screening pass: the largest |G|
must be the reported power and sit at the reported cell.

Shapes at the edges of the pass: one and two blocks of 16 operand rows, IFs
that split evenly by the parity of their lattice position and ones that do
not, a single IF (every MBD bin alike), compact lattices (coarse MBD grids of
1 to 8 tiles) and spread ones, every channel count, the smallest and largest
unit counts; rates that fill the blocks of eight tasks evenly and ones that do
not, windows shorter and longer than the ring of spectra.  Data at the edges of its
bound: noise with one overwhelming channel (many near-equal units), one
overwhelming sample, zeros, magnitudes at both ends of float32, and NaN and
infinite samples.

Tolerance: the dumped and the searched cells are separate compilations of the
same float32 sums (4e-6 relative in power where multiply-adds fuse
differently); the search keeps 19 mantissa bits of |G|^2 for the choice of the
cell."""
import numpy as np
import pytest
import torch

from paper_1801_02391_amd import frbx
from paper_1801_02391_amd import workloads as W

from gpu_helpers import note

pytestmark = pytest.mark.gpu

POWER_TOL = 4e-6
N_DM = 80   # enough segments (4096) for a search to be screened
CELL_TOL = 2.0 ** -18 + 2 * POWER_TOL

VGOS = [b + 32.0 * i for b in (3000.0, 5240.0, 6360.0, 10200.0) for i in range(8)]
LATTICES = {
    "1if": [3000.0],
    "3if-spread": [3000.0, 3032.0, 5240.0],
    "16if-compact": [3000.0 + 32.0 * i for i in range(16)],
    "9if-compact": [3000.0 + 32.0 * i for i in range(9)],
    "5if-compact": [3000.0 + 32.0 * i for i in (0, 1, 2, 3, 6)],
    "17if": VGOS[:17],
    "20if-even": [3000.0 + 64.0 * i for i in range(19)] + [3032.0],   # 19 even positions, 1 odd
    "32if-vgos": VGOS,
}


def _search(f0, J, P, R, precision, V, windows, t_ap=1.0):
    lay = dict(n_baselines=V.shape[0], if_freq_mhz=f0, n_if=len(f0), n_chan=J, chan_bw_mhz=32.0 / J, t_ap_ms=t_ap,
               n_frames=V.shape[-1])
    s = frbx.Search(lay)
    s.configure(dict(dm_lo=0.0, dm_step=0.5, n_dm=N_DM, sbd_pad=P, n_mbd=256, n_rate=R, windows=windows, threshold=3.0,
                     n_win_min=1, n_bl_min=1, precision=precision))
    s.load(torch.from_numpy(V).to("cuda:0"))
    s.run()
    return s


def _noise(N, J, K, seed):
    g = np.random.default_rng(seed)
    return (g.standard_normal((1, N, J, K)) + 1j * g.standard_normal((1, N, J, K))).astype(np.complex64)


def _check(s, windows, n_check=14):
    """Power and cell of segments spread over every window against the dump."""
    P, I = s.power_cube()
    seg = s.segments()
    off = np.cumsum([0] + seg["n_seg"])
    for wi in range(len(windows)):
        for q in np.unique(np.linspace(0, seg["n_seg"][wi] - 1, n_check).astype(int)):
            for d in (0, N_DM - 1):
                p, i = float(P[0, d, off[wi] + q]), int(I[0, d, off[wi] + q])
                g2 = s.dump_segment(0, d, wi, int(q)).reshape(-1).astype(np.float64)
                top = np.sqrt(g2.max())
                assert abs(p - top) <= POWER_TOL * top, (wi, q, d, p, top)
                assert g2[i] >= g2.max() * (1 - CELL_TOL), (wi, q, d, i, int(g2.argmax()))


@pytest.mark.parametrize("precision", ["f32", "f16x3", "f16"])
@pytest.mark.parametrize("name,J,P,R", [("1if", 32, 4, 2), ("3if-spread", 64, 1, 4), ("16if-compact", 32, 8, 2),
                                        ("17if", 32, 2, 4), ("20if-even", 64, 2, 3), ("32if-vgos", 64, 4, 8),
                                        ("32if-vgos", 32, 4, 9), ("32if-vgos", 16, 4, 4), ("32if-vgos", 128, 4, 3),
                                        ("20if-even", 128, 1, 2), ("16if-compact", 256, 4, 2), ("3if-spread", 256, 1, 1),
                                        ("9if-compact", 64, 4, 4), ("5if-compact", 16, 8, 3),
                                        ("32if-vgos", 64, 4, 5), ("17if", 64, 1, 11), ("20if-even", 128, 2, 4),
                                        ("32if-vgos", 128, 4, 9), ("3if-spread", 128, 4, 6),
                                        ("16if-compact", 256, 4, 4), ("3if-spread", 256, 2, 13)])
def test_screened_peak_is_the_largest_cell(name, J, P, R, precision):
    f0, windows = LATTICES[name], [1, 2, 5]
    note(f"screen {name} J={J} P={P} R={R} {precision}")
    V = _noise(len(f0), J, 70, 7)
    _check(_search(f0, J, P, R, precision, V, windows), windows, 8)


@pytest.mark.parametrize("precision", ["f32", "f16"])
@pytest.mark.parametrize("kind", ["channel", "sample", "tiny", "huge"])
def test_screened_peak_of_extreme_data(kind, precision):
    f0, windows, J = LATTICES["17if"], [2, 4], 32
    note(f"screen data {kind} {precision}")
    V = _noise(len(f0), J, 60, 11)
    if kind == "channel":
        V[:, 3, 9] *= 300.0
    elif kind == "sample":
        V[:, 2, 5, 30] *= 1e6
    elif kind == "tiny":
        V *= np.float32(1e-14)
    else:
        V *= np.float32(1e13)
    _check(_search(f0, J, 4, 3, precision, V, windows), windows)


@pytest.mark.parametrize("precision", ["f32", "f16x3", "f16"])
def test_screened_search_of_zeros_and_non_finite_samples(precision):
    """All-zero segments have power 0 at the first cell searched (float32:
    packed index 0; the matrix-core forms: the first cell of the first unit,
    SBD bin PJ / 2); segments with a NaN or infinite sample are not finite and
    the others are untouched."""
    f0, windows, J = LATTICES["17if"], [2, 4], 32
    note(f"screen zeros / non-finite {precision}")
    V = _noise(len(f0), J, 80, 13)
    V[..., 20:40] = 0.0
    s = _search(f0, J, 4, 3, precision, V, windows)
    P, I = s.power_cube()
    mid = I[0, 0, 24:30]   # DM 0: window 2, segments inside the zero stretch
    assert np.all(P[0, 0, 24:30] == 0.0) and np.all(mid == (0 if precision == "f32" else 4 * J // 2 * 256))
    W_ = V.copy()
    W_[0, 4, 6, 60] = np.nan
    W_[0, 1, 7, 10] = np.inf
    Pn, In = _search(f0, J, 4, 3, precision, W_, windows).power_cube()
    seg = s.segments()
    k0 = np.concatenate([np.arange(n) * h for n, h in zip(seg["n_seg"], seg["hop"])])   # DM 0: the segments' APs
    k1 = k0 + np.repeat(windows, seg["n_seg"]) - 1
    hit = np.zeros(P.shape[2], dtype=bool)
    for k in (10, 60):
        hit |= (k0 <= k) & (k1 >= k)
    assert np.array_equal(~np.isfinite(Pn[0, 0]), hit)
    if precision == "f32":   # (the float16 operand scale follows the largest finite component)
        assert np.array_equal(Pn[0, 0, ~hit], P[0, 0, ~hit]) and np.array_equal(In[0, 0, ~hit], I[0, 0, ~hit])


@pytest.mark.parametrize("name,J", [("5if-compact", 16), ("16if-compact", 32), ("9if-compact", 64), ("17if", 16),
                                    ("3if-spread", 32), ("32if-vgos", 64)])
def test_segments_with_few_and_with_all_cells_alike(name, J):
    """Noise first (a few candidates per segment, evaluated one by one), then
    one channel only, where |G| is the same in every SBD bin and a segment is
    searched as a whole: the segments of one tile go both ways."""
    f0, windows = LATTICES[name], [1, 3]
    note(f"screen alike {name} J={J}")
    V = _noise(len(f0), J, 70, 17)
    V[:, :, : J // 2 + 1, 35:] = 0.0
    V[:, :, J // 2 + 2 :, 35:] = 0.0
    s = _search(f0, J, 4, 3, "f32", V, windows)
    _check(s, windows)
    P, I = s.power_cube()
    p, i = torch.empty(P.size, device="cuda:0"), torch.empty(P.size, dtype=torch.int32, device="cuda:0")
    assert s.run_cube_noalloc(p, i) == P.size
    torch.cuda.synchronize()
    assert np.array_equal(p.cpu().numpy(), P.ravel()) and np.array_equal(i.cpu().numpy(), I.ravel())
