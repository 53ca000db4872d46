"""Source maps and histograms at the edges of the smoothing kernels' tiles
against the FP64 oracle: 1 to 8 outputs a thread, rows of 256 outputs, taps
in chunks of 256, radii up to and beyond the ones whose taps fit in LDS, and
the disk's prefix sums."""
import numpy as np
import pytest

from oracle import light_curves as OL
from oracle import surrogate as OS
from paper_1703_09707_amd import raysh as R
from paper_1703_09707_amd import surrogate as S

pytestmark = pytest.mark.gpu

RTOL = 1e-13   # as in the other source-map tests: exp() may differ by an ulp, the sums run in the same order


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _counts(torch, nx, ny, seed, hi=200):
    c = np.random.default_rng(seed).integers(0, hi, (ny, nx)).astype(np.int32)
    return c, torch.from_numpy(c).cuda()


# nx, ny, pixel sizes, source size: radii (rx, ry) in the comment
@pytest.mark.parametrize("nx,ny,px,py,size", [
    (3, 4, 1.0, 1.0, 0.2),                # (1, 1), 1 x 2 outputs are too few: widened below
    (100, 90, 1.0, 1.0, 1.0),             # (3, 3), 4 outputs a thread
    (400, 407, 1.0, 1.0, 2.0),            # (6, 6)
    (600, 507, 1.0, 1.0, 2.5),            # (8, 8)
    (800, 709, 1.0, 1.0, 1.3),            # (4, 4), 8, ragged in both directions
    (300, 30, 0.1, 1.0, 4.23),            # (127, 13): 255 taps along a row
    (300, 40, 0.1, 1.0, 4.26),            # (128, 13): 257
    (1100, 40, 0.01, 1.0, 1.7065),        # (512, 6): the last in LDS
    (1100, 40, 0.01, 1.0, 1.7073),        # (513, 6): beyond
    (40, 1100, 1.0, 0.01, 1.7065)])       # (6, 512)
def test_gaussian_tiles_match_oracle(torch, nx, ny, px, py, size):
    if nx == 3:
        nx, ny = 5, 6
    host, counts = _counts(torch, nx, ny, nx * 1009 + ny)
    pix = (0.0, 0.0, px, py, nx, ny)
    mu, grid = R.source_map(counts, pix, 0.37, "gaussian", size)
    want = OL.source_map(host, 0.37, R.SOURCE_GAUSSIAN, size, px, py)
    assert tuple(mu.shape) == want.shape
    np.testing.assert_allclose(mu.cpu().numpy(), want, rtol=RTOL, atol=0)
    # the histogram's passes: the same smoothing, binned
    for nbins in (1, 64, 4096):
        hist = S.Histogrammer(nx, ny)
        bins, h = hist(counts, 0.37, size, px, py, 37.0, nbins=nbins)
        lm_h, lm_c, frac = OS.log_mag_histogram(host, 0.37 * px, py, px, py, size, 37.0, nbins=nbins)
        near = int(np.count_nonzero(frac < 1e-9))
        got = bins.cpu().numpy().astype(np.int64)
        assert got.sum() == want.size
        assert np.abs(got - lm_c).sum() <= 2 * near
        np.testing.assert_array_equal(h.cpu().numpy(), (got / got.sum()).astype(np.float32))
        bins2, _ = hist(counts, 0.37, size, px, py, 37.0, nbins=nbins, out=(torch.empty_like(bins), None))
        np.testing.assert_array_equal(bins2.cpu().numpy(), got)


@pytest.mark.parametrize("nx,ny,px,py,size", [
    (3, 3, 1.0, 1.0, 0.3), (64, 257, 1.0, 1.0, 1.0), (64, 257, 1.0, 1.0, 3.9), (65, 257, 1.0, 1.0, 4.0), (255, 61, 1.0, 1.0, 5.5), (256, 64, 0.5, 1.0, 6.0),
    (257, 70, 1.0, 0.25, 3.2), (30, 300, 1.0, 0.01, 0.9), (1025, 33, 0.05, 1.0, 14.9), (40, 513, 1.0, 0.07, 13.3)])
def test_disk_prefix_sums_match_oracle_exactly(torch, nx, ny, px, py, size):
    """Counts up to 2^31 - 1 and down to -2^31: the sums are exact in 64 bits."""
    c = np.random.default_rng(nx * 31 + ny).integers(-2 ** 31, 2 ** 31, (ny, nx)).astype(np.int32)
    counts = torch.from_numpy(c).cuda()
    mu, _ = R.source_map(counts, (0.0, 0.0, px, py, nx, ny), 0.37, "disk", size)
    want = OL.source_map(c, 0.37, R.SOURCE_DISK, size, px, py)
    np.testing.assert_array_equal(mu.cpu().numpy(), want)
