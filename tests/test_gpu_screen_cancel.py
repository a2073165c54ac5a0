"""Windows whose APs cancel: an interference that alternates in sign from AP
to AP, far above the noise, leaves segment sums that are small beside the
spectra they are formed from, and the float32 rounding of the sums (which
scales with the spectra) is of the noise's own size.  The screened search must
report what the search of every cell reports, bit for bit.

The same spectra are searched at one DM trial of step 0 (few segments: every
cell is evaluated) and at as many equal trials as it takes to be screened."""
import numpy as np
import pytest
import torch

from paper_1801_02391_amd import frbx

from gpu_helpers import note

pytestmark = pytest.mark.gpu

VGOS = [b + 32.0 * i for b in (3000.0, 5240.0, 6360.0, 10200.0) for i in range(8)]


def _cube(f0, J, R, windows, V, n_dm):
    s = frbx.Search(dict(n_baselines=1, if_freq_mhz=f0, n_if=len(f0), n_chan=J, chan_bw_mhz=32.0 / J, t_ap_ms=1.0,
                         n_frames=V.shape[-1]))
    # (a rate step so fine that every rate leaves the cancellation)
    s.configure(dict(dm_lo=0.0, dm_step=0.0, n_dm=n_dm, sbd_pad=4, n_mbd=256, n_rate=R, rate_step=1e-16, windows=windows,
                     threshold=3.0, n_win_min=1, n_bl_min=1, precision="f32"))
    s.load(torch.from_numpy(V).to("cuda:0"))
    s.run()
    return s.power_cube()


@pytest.mark.parametrize("amp", [1e5, 1e7])
@pytest.mark.parametrize("name,f0,J,R,windows", [("ring", VGOS, 64, 8, [2, 4]), ("no ring", VGOS[:17], 32, 8, [2, 6]),
                                                 ("one row block", VGOS[:16], 32, 8, [2, 8]),
                                                 ("few rows", VGOS[:5], 16, 4, [2, 4])])
def test_cancelling_windows_keep_the_searchs_bits(name, f0, J, R, windows, amp):
    note(f"screen cancel {name} {amp:g}")
    g, K, N = np.random.default_rng(5), 100, len(f0)
    V = g.standard_normal((1, N, J, K)) + 1j * g.standard_normal((1, N, J, K))
    V = V + amp * np.exp(2j * np.pi * g.random((1, N, J, 1))) * (1 - 2 * (np.arange(K) % 2))
    V = V.astype(np.complex64)
    P1, I1 = _cube(f0, J, R, windows, V, 1)
    assert P1.shape[2] * R < 4096
    n_dm = -(-4096 // (P1.shape[2] * R))
    P2, I2 = _cube(f0, J, R, windows, V, 2 * n_dm)
    assert np.array_equal(P2, np.broadcast_to(P1, P2.shape)) and np.array_equal(I2, np.broadcast_to(I1, I2.shape))
