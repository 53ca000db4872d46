"""Light curves by waves of 256 samples where every sample of a wave lies
inside the map and where some do not: tracks along the edges, one rounding
step beyond them, of one point, off the map and not finite; chunks cut by 1 to
63 samples; maps of 2 pixels a side and of 2^24 columns (64-bit addresses)."""
import numpy as np
import pytest

from oracle import light_curves as OL
from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _tracks(nx, ny, seed):
    """End points in units of pixels on a grid whose centres are the integers."""
    w, h = nx - 1.0, ny - 1.0
    up = np.nextafter
    rows = [(0, 0, w, h), (w, h, 0, 0), (0, h, w, h), (w, 0, w, h), (0, 0, w, 0),          # corners and edges
            (0, up(h, 2 * h), w, h), (up(0, -1), 0, 0, h), (0, 0, up(w, 2 * w), h),        # one step beyond
            (w / 2, h / 2, w / 2, h / 2), (w, h, w, h), (0.5, 0.5, 0.5, 0.5),              # points
            (-3, h / 2, w + 3, h / 2), (w / 2, -2, w / 2, h / 2), (-5, -5, -1, -1),        # in and out
            (np.nan, 0, w, h), (0, 0, np.inf, h), (0, -np.inf, w, h), (0, 0, 1e300, 1e300), (1e308, 0, -1e308, h)]
    rng = np.random.default_rng(seed)
    a = np.array(rows + [tuple(r) for r in rng.uniform(-0.1, 1.1, (60, 4)) * [w, h, w, h]], float)
    return [np.ascontiguousarray(a[:, c]) for c in range(4)]


def _check(torch, mu, host, grid, tracks, n_samples):
    dev = [torch.from_numpy(t).cuda() for t in tracks]
    with np.errstate(all="ignore"):
        want = OL.light_curves(host, grid, *tracks, n_samples)
    plain = R.light_curves(mu, grid, *dev, n_samples).cpu().numpy()
    np.testing.assert_array_equal(plain, want)
    order, srt = R.track_order(grid, *dev, sorted_end_points=True)
    np.testing.assert_array_equal(R.light_curves(mu, grid, *dev, n_samples, order=order, sorted=srt).cpu().numpy(),
                                  want)


@pytest.mark.parametrize("n_samples", [64, 65, 127, 200, 255, 256, 257, 319, 512, 700])
@pytest.mark.parametrize("nx,ny", [(2, 2), (2, 90), (75, 2), (61, 130)])
def test_chunks(torch, nx, ny, n_samples):
    host = np.random.default_rng(nx).uniform(0.1, 9.0, (ny, nx))
    _check(torch, torch.from_numpy(host).cuda(), host, (-0.5, -0.5, 1.0, 1.0, nx, ny), _tracks(nx, ny, n_samples),
           n_samples)


@pytest.mark.parametrize("nx", [(1 << 24) - 1, 1 << 24])
def test_long_rows(torch, nx):
    """The last row length of the 32-bit addresses, and the first beyond."""
    ny, n_samples = 3, 300
    mu = (torch.arange(nx * ny, dtype=torch.float64, device="cuda").view(ny, nx) % 1013) * 0.37
    _check(torch, mu, mu.cpu().numpy(), (-0.5, -0.5, 1.0, 1.0, nx, ny), _tracks(nx, ny, 1), n_samples)
