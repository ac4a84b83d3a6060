"""GPU: spectral statistics and peaks at the ends of the kernels' layouts (bins
held on chip up to 4096, 16 bins and 256 probes at a time), against the oracle."""
import numpy as np
import pytest

from oracle import spectra as OS
from paper_0809_1547_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,K", [(1, 1), (1, 3), (63, 15), (64, 16), (65, 17), (255, 257), (256, 33), (257, 31),
                                 (3, 4095), (3, 4096), (3, 4097), (600, 5000)])
def test_stats_and_peaks_match_oracle(P, K):
    from paper_0809_1547_amd import mbf
    F, om = I.synthetic_spectra(P, K, seed=K, lines=((0.45, 0.03, 1.0), (0.7, 0.02, 0.6), (0.2, 0.05, 0.3)))
    F = F * (1.0 + 0.01 * np.sin(np.arange(K) * 1.7))         # ripples: more candidates than lines
    spec = np.stack([F.real, F.imag], -1)
    got, want = mbf.mbf_spectral_stats(spec, om, 0.5), OS.spectral_stats(F, om, 0.5)
    for key in ("peak_bin", "fit_lo", "fit_hi", "fit_ok"):
        assert got[key] == want[key], key
    for key in ("total", "peak_value", "mean_omega", "std_omega"):
        assert got[key] == pytest.approx(want[key], rel=1e-9), key
    for rel, top in ((0.05, 8), (0.0, 40), (1.0, 3)):
        assert list(mbf.mbf_spectral_peaks(spec, min_rel=rel, max_peaks=top)) == list(OS.spectral_peaks(F, rel, top))
