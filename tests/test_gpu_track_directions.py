"""raysh_track_order where it also sorts a cell's tracks by direction: from 16
tracks a cell on, over one to 65536 counters and the scan's workgroups of
2048, with tracks of no length, of one point far off the map, and NaN."""
import numpy as np
import pytest

from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu

DIRECTIONS = 16


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _cells(grid, tracks):
    """Morton number of each track's cell (16 x 16 pixels)."""
    x0, y0, px, py, nx, ny = grid
    out = np.zeros(len(tracks[0]), np.int64)
    for axis, (a, b, o, p, n) in enumerate(((tracks[0], tracks[2], x0, px, nx), (tracks[1], tracks[3], y0, py, ny))):
        cells = (n + 15) // 16
        with np.errstate(invalid="ignore"):
            c = ((0.5 * (a + b) - o) * (1.0 / p)) / 16.0
            c = np.where(c >= 0, np.minimum(np.nan_to_num(c, nan=0.0, posinf=cells), cells - 1), 0).astype(np.int64)
        for bit in range(12):
            out |= ((c >> bit) & 1) << (2 * bit + axis)
    return out


@pytest.mark.parametrize("nx,ny,n", [(16, 16, 15), (16, 16, 16), (16, 16, 5000), (40, 33, 255), (40, 33, 256),
                                     (40, 33, 257), (200, 30, 4096), (512, 512, 16383), (512, 512, 16384),
                                     (530, 512, 70001), (1024, 1024, 300_001)])
def test_direction_order(torch, nx, ny, n):
    grid = (-5.0, -4.0, 10.0 / nx, 8.0 / ny, nx, ny)
    rng = np.random.default_rng(n)
    mx, my = rng.uniform(-5.2, 5.2, n), rng.uniform(-4.2, 4.2, n)
    ang, half = rng.uniform(0, 2 * np.pi, n), rng.uniform(0.01, 0.5, n)
    half[::7] = 0.0                      # no length
    tracks = [mx - half * np.cos(ang), my - half * np.sin(ang), mx + half * np.cos(ang), my + half * np.sin(ang)]
    tracks[0][1 % n], tracks[3][2 % n], tracks[1][3 % n] = 1e300, np.nan, -np.inf
    dev = [torch.from_numpy(a).cuda() for a in tracks]
    order, srt = R.track_order(grid, *dev, sorted_end_points=True)
    o = order.cpu().numpy()
    assert np.array_equal(np.sort(o), np.arange(n))
    assert np.array_equal(srt.cpu().numpy(), np.stack([a[o] for a in tracks]), equal_nan=True)
    cells = _cells(grid, tracks)[o]
    assert np.all(np.diff(cells) >= 0)
    side = max((nx + 15) // 16, (ny + 15) // 16)
    keys = (1 << int(np.ceil(np.log2(side)))) ** 2
    if n < keys * DIRECTIONS:
        return
    # within a cell, directions come bin after bin
    dx, dy = (tracks[2] - tracks[0]) / grid[2], (tracks[3] - tracks[1]) / grid[3]
    with np.errstate(invalid="ignore"):
        along = np.where(dy < 0, -dx, dx) / (np.abs(dx) + np.abs(dy))
    d = ((1 - along) * (DIRECTIONS / 2))[o]
    ok = np.isfinite(d)
    d, c = d[ok], cells[ok]
    for cell in np.unique(c):
        v = d[c == cell]
        assert np.all(np.maximum.accumulate(v) - v <= 1.0 + 1e-4)   # a bin's width, and its edges in 32 bits


def test_curves_of_directed_order(torch):
    """The curves are the same with the order as without it, for a number of
    workgroups that is and one that is not a multiple of the XCDs."""
    rng = np.random.default_rng(5)
    mu = torch.from_numpy(rng.uniform(0.1, 5.0, (160, 150))).cuda()
    grid = (-1.0, -1.0, 2.0 / 150, 2.0 / 160, 150, 160)
    for n in (4096, 4103, 5):
        a = [torch.from_numpy(rng.uniform(-1.05, 1.05, n)).cuda() for _ in range(4)]
        for samples in (70, 200):
            plain = R.light_curves(mu, grid, *a, samples)
            order, srt = R.track_order(grid, *a, sorted_end_points=True)
            got = R.light_curves(mu, grid, *a, samples, order=order, sorted=srt)
            assert torch.equal(torch.isnan(plain), torch.isnan(got))
            assert torch.equal(torch.nan_to_num(plain), torch.nan_to_num(got))
