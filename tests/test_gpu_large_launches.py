"""GPU: analyses with more bins or frequencies than one launch of their tiled
kernels may hold (2^32 threads along a side)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_power_of_more_bins_than_a_tiled_launch_holds():
    import torch
    from paper_0809_1547_amd import mbf
    K = (1 << 26) + 1000
    spec = torch.zeros((1, K, 2), dtype=torch.float64, device="cuda")
    at = [3, 1 << 26, K - 2]
    for q, k in enumerate(at):
        spec[0, k, q % 2] = 2.0 + q
    got = mbf.mbf_spectral_peaks(spec, min_rel=0.0, max_peaks=8)
    assert list(got) == at[::-1]
