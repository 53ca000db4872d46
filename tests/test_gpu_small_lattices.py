"""One-pass FP64 on lattices that do not fill the device in the default shape:
the workgroup's waves share a tile and split the stars.  Against the oracle
ray by ray, and against the one-pass shape itself, at the edges of the tiles
(64 x 32, 32 x 32, 32 x 16 and 16 x 16 rays) and of the stars' runs (4, 8 and
16 waves)."""
import numpy as np
import pytest

from oracle import shooter as ora
from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu

BETA_TOL = 1e-12   # of the error scale S: the FP64 bar of the one-pass tests
PIX = (-0.9, -0.8, 1.7 / 45, 1.9 / 52, 45, 52)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _rays(nx, ny, i0=0, j0=0):
    return (-1.25, -1.25, 2.5 / max(nx, ny), 2.5 / max(nx, ny), nx, ny, i0, j0)


def _lens(n, on_ray=None, seed=0):
    rng = np.random.default_rng(1000 + n + seed)
    xs, ys, ms = rng.uniform(-3, 3, n), rng.uniform(-3, 3, n), rng.uniform(0.01, 0.05, n)
    if on_ray is not None and n:
        xs[n // 2], ys[n // 2] = on_ray
    return (0.1, 0.1, -0.05, xs, ys, ms)


def _theta(rays, i, j):
    return (float(rays[0] + ((rays[6] + i) + 0.5) * rays[2]), float(rays[1] + ((rays[7] + j) + 0.5) * rays[3]))


def _edge(bx, by, s, pix):
    """Rays within the beta bar of a pixel edge: either pixel is right."""
    with np.errstate(invalid="ignore"):
        u, v = (bx - pix[0]) / pix[2], (by - pix[1]) / pix[3]
        near = (np.abs(u - np.round(u)) * pix[2] <= BETA_TOL * s) | (np.abs(v - np.round(v)) * pix[3] <= BETA_TOL * s)
    return near


def _check(ctx, lens, rays, pix):
    gx, gy, gb = (t.cpu().numpy() for t in ctx.shoot(rays, "fp64", pix))
    ox, oy, ob = ora.shoot(lens, rays, pix)
    s = ora.error_scale_block(lens, rays)
    fin = np.isfinite(ox) & np.isfinite(oy)
    assert np.array_equal(fin, np.isfinite(gx) & np.isfinite(gy))
    assert np.all(np.abs(gx[fin] - ox[fin]) <= BETA_TOL * s[fin])
    assert np.all(np.abs(gy[fin] - oy[fin]) <= BETA_TOL * s[fin])
    near = _edge(ox, oy, s, pix)
    assert np.count_nonzero((gb != ob) & ~near) == 0
    # the map is the histogram of the same bins
    m, n = ctx.map(rays, pix, "fp64", n_binned=True)
    ok = gb[gb >= 0]
    assert np.array_equal(m.cpu().numpy().ravel(), np.bincount(ok, minlength=pix[4] * pix[5]))
    assert int(n) == ok.size
    return gx, gy, gb, s, near


@pytest.mark.parametrize("nx,ny", [(1, 1), (15, 17), (16, 16), (33, 31), (250, 130), (256, 257), (333, 200), (500, 490),
                                   (640, 700), (1025, 289), (1, 3000), (2049, 3)])
@pytest.mark.parametrize("n_stars", [0, 1, 3, 15, 16, 17, 333])
def test_shared_tiles_match_oracle(torch, nx, ny, n_stars):
    rays = _rays(nx, ny, 3, 1)
    lens = _lens(n_stars, _theta(rays, nx // 2, ny // 3))
    with R.Context(lens) as ctx:
        gx, gy, gb, s, near = _check(ctx, lens, rays, PIX)
        ctx.set_tile("fp64", 8, 4, 16, 1)   # the one-pass form
        px, py, pb = (t.cpu().numpy() for t in ctx.shoot(rays, "fp64", PIX))
    fin = np.isfinite(px) & np.isfinite(py)
    assert np.array_equal(fin, np.isfinite(gx) & np.isfinite(gy))
    assert np.all(np.abs(gx[fin] - px[fin]) <= BETA_TOL * s[fin])
    assert np.all(np.abs(gy[fin] - py[fin]) <= BETA_TOL * s[fin])
    assert np.count_nonzero((gb != pb) & ~near) == 0


@pytest.mark.parametrize("pix", [(0.0, -0.7, 0.1, 0.1, 8, 14),            # X0 = 0: the division
                                 (-0.8, -0.7, 2.0 ** -301, 0.1, 4, 14),   # a pixel below the fast form's range
                                 (-0.8, -0.7, 1e-3, 3e-3, 1600, 467),     # counts beyond the LDS window
                                 (50.0, 50.0, 0.1, 0.1, 7, 7)])           # no ray
def test_windows(torch, pix):
    for nx, ny, n in ((200, 160, 40), (700, 640, 40)):
        lens, rays = _lens(n), _rays(nx, ny)
        with R.Context(lens) as ctx:
            _check(ctx, lens, rays, pix)


def test_wide_separations(torch):
    """Separations whose shared product leaves FP64's range: those rays are
    summed again with a division per star, within each wave's run."""
    for spread in (1e30, 1e-30):
        lens = _lens(37)
        lens = lens[:3] + (lens[3] * spread, lens[4] * spread, lens[5])
        rays = tuple(v * spread for v in _rays(90, 70)[:4]) + (90, 70, 0, 0)
        pix = tuple(v * spread for v in PIX[:4]) + PIX[4:]
        with R.Context(lens) as ctx:
            _check(ctx, lens, rays, pix)


def test_captured_map(torch):
    """The allocation-free one-pass map in a graph, replayed between eager
    calls, gives the eager map each time."""
    lens, rays = _lens(120), _rays(400, 300)
    with R.Context(lens) as ctx:
        want = ctx.map(rays, PIX, "fp64")
        counts = torch.zeros_like(want)
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        ctx.set_stream(side)
        ctx.map_split_noalloc(rays, PIX, 1, counts)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            counts.zero_()
            ctx.map_split_noalloc(rays, PIX, 1, counts)
        torch.cuda.synchronize()
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(counts, want)
            again = torch.zeros_like(want)
            torch.cuda.synchronize()
            ctx.map(rays, PIX, "fp64", counts=again)
            torch.cuda.synchronize()
            assert torch.equal(again, want)
