"""GPU: spectral power of few probes and of many bins (a thread a bin) beside the
workgroups that share a bin's probes, and peaks among many candidates, few and
many asked for, against the oracle."""
import numpy as np
import pytest

from oracle import spectra as OS

pytestmark = pytest.mark.gpu


def _noise(P, K):
    rng = np.random.default_rng(P * 100003 + K)
    F = rng.standard_normal((P, K)) + 1j * rng.standard_normal((P, K))
    return F * (1.0 + 20.0 * np.exp(-((np.arange(K) / K - 0.5) / 0.02) ** 2))


@pytest.mark.parametrize("P,K", [(1, 874), (8, 63), (8, 65), (9, 64), (17, 874), (3, 32767), (3, 32768), (20, 40001)])
def test_power_kernels_agree_with_oracle(P, K):
    from paper_0809_1547_amd import mbf
    F = _noise(P, K)
    om = np.linspace(1.0, 2.0, K)
    spec = np.stack([F.real, F.imag], -1)
    got, want = mbf.mbf_spectral_stats(spec, om, 0.5), OS.spectral_stats(F, om, 0.5)
    assert got["peak_bin"] == want["peak_bin"]
    for key in ("total", "peak_value", "mean_omega", "std_omega"):
        assert got[key] == pytest.approx(want[key], rel=1e-9), key


@pytest.mark.parametrize("K", [30, 257, 874, 1500])
@pytest.mark.parametrize("top", [1, 2, 7, 16, 200, 1024])
def test_peaks_among_many_candidates(K, top):
    from paper_0809_1547_amd import mbf
    F = _noise(2, K)
    F[:, 5] = F[:, 9] = F[:, 7] * 0.5                  # equal values
    spec = np.stack([F.real, F.imag], -1)
    assert list(mbf.mbf_spectral_peaks(spec, min_rel=0.0, max_peaks=top)) == list(OS.spectral_peaks(F, 0.0, top))
