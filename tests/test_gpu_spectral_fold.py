"""The fused spectral kernel's folded frames at the edges of its tiles: odd
and even sizes (a middle row or column is its own mirror), sizes read in
16-byte chunks and one by one, quadrants of one to four row tiles, partial and
full column tiles, and the sizes just past it (the general path); a NaN or an
infinity in a frame reaches every band of that frame's lag."""
import numpy as np
import pytest

import oracle

from test_gpu_spectral import CORR_ABS, gpu_corr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,bands", [
    (1, 16, 2), (2, 1, 1), (3, 3, 2), (31, 33, 5), (32, 32, 6), (33, 24, 5), (15, 100, 8), (17, 128, 8), (63, 127, 12),
    (64, 121, 12), (65, 64, 9), (72, 128, 24), (96, 98, 16), (97, 50, 10), (128, 40, 10), (128, 65, 12),
    (129, 16, 6), (16, 130, 6),
])
def test_fold_edges(H, W, bands):
    """Within the bar of the other spectral tests; fp32 transforms whose sums are half as long are no further off."""
    lat = np.random.default_rng(H * 1000 + W).standard_normal((2, 4, H, W)).astype(np.float32)
    band = np.random.default_rng(1).integers(0, bands, (H, W)).astype(np.int32)
    got = gpu_corr(lat, band, bands, 3)
    with np.errstate(invalid="ignore", divide="ignore"):
        import warnings
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            ref = oracle.band_correlations(lat, band, bands, 3)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    ok = ~np.isnan(ref)
    assert np.abs(got[ok] - ref[ok]).max(initial=0.0) <= CORR_ABS, np.abs(got[ok] - ref[ok]).max()


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("place", [(10, 12), (0, 3), (10, 3), (20, 24)])
def test_non_finite_values_reach_every_band(value, place):
    H, W, bands = 21, 25, 4  # (10, 12) is the middle of both directions
    lat = np.random.default_rng(3).standard_normal((1, 4, H, W)).astype(np.float32)
    lat[0, 2][place] = value
    band = np.full((H, W), -1, np.int32)
    for k in range(bands):  # band k holds one parity of rows and columns only
        band[k // 2::2, k % 2::2] = k
    got = gpu_corr(lat, band, bands, 3)
    assert np.isnan(got[:, 2]).all()
    assert np.isfinite(got[:, [0, 1, 3]]).all()
