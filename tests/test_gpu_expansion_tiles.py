"""The expansion mode's tile kernel where it can go wrong: each tile shape
(64 / 2^k by 64 * 2^k rays) with ragged edges, one tile and four tiles a
workgroup, near lists within and beyond a tile's 256 and a block's 4 * 512
stars, a ray exactly on a star, and windows that take the division or its
five-instruction form.  Rays are checked one by one against the FP64 oracle;
every pixel is checked against IEEE division of the kernel's own beta."""
import numpy as np
import pytest

from oracle import shooter as ora
from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu

BETA_TOL = 1e-12   # of the error scale S: the FP64 bar of the other expansion tests


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _ieee_bins(bx, by, pix):
    """Algorithm 1's pixel step on given beta, in NumPy's IEEE arithmetic."""
    X0, Y0, Px, Py, NX, NY = pix
    with np.errstate(invalid="ignore", over="ignore"):
        u, v = (bx - X0) / Px, (by - Y0) / Py
        ok = np.isfinite(bx) & np.isfinite(by) & (u >= 0) & (u < NX) & (v >= 0) & (v < NY)
    out = np.full(bx.shape, -1, np.int64)
    out[ok] = np.floor(v[ok]).astype(np.int64) * NX + np.floor(u[ok]).astype(np.int64)
    return out


def _check(torch, ctx, lens, rays, pix, sample=None):
    """Per-ray outputs against the oracle (all rays, or `sample` of them),
    bins against IEEE division, and the map against the bins."""
    gx, gy, gb = (t.cpu().numpy() for t in ctx.shoot(rays, "fp64_expansion", pix))
    nx, ny = rays[4], rays[5]
    if sample is None:
        ox, oy, _ = ora.shoot(lens, rays, pix)
        s = ora.error_scale_block(lens, rays)
        hx, hy = gx, gy
    else:
        rng = np.random.default_rng(nx + ny)
        ii, jj = rng.integers(0, nx, sample), rng.integers(0, ny, sample)
        ii[:4], jj[:4] = (0, nx - 1, 0, nx - 1), (0, 0, ny - 1, ny - 1)
        ox, oy, _ = ora.shoot_list(lens, rays, pix, ii, jj)
        tx, ty = ora.image_angles(rays)
        s = ora.error_scale(lens, tx[ii], ty[jj])
        hx, hy = gx[jj, ii], gy[jj, ii]
    fin = np.isfinite(ox) & np.isfinite(oy)
    assert np.array_equal(fin, np.isfinite(hx) & np.isfinite(hy))
    assert np.all(np.abs(hx[fin] - ox[fin]) <= BETA_TOL * s[fin])
    assert np.all(np.abs(hy[fin] - oy[fin]) <= BETA_TOL * s[fin])
    want = _ieee_bins(gx, gy, pix)
    assert np.array_equal(gb.astype(np.int64), want)
    counts, n = ctx.map(rays, pix, "fp64_expansion", n_binned=True)
    hist = np.bincount(want[want >= 0], minlength=pix[4] * pix[5])
    assert np.array_equal(counts.cpu().numpy().ravel().astype(np.int64), hist)
    assert int(n) == int(hist.sum())


def _lens(seed, n, spread, on_ray=None, cluster=0, radius=0.05):
    rng = np.random.default_rng(seed)
    xs, ys = rng.uniform(-spread, spread, n), rng.uniform(-spread, spread, n)
    ms = rng.uniform(0.01, 0.05, n)
    if cluster:
        r, phi = radius * np.sqrt(rng.random(cluster)), 2 * np.pi * rng.random(cluster)
        xs, ys = np.concatenate([xs, r * np.cos(phi)]), np.concatenate([ys, r * np.sin(phi)])
        ms = np.concatenate([ms, rng.uniform(1e-4, 2e-4, cluster)])
    if on_ray is not None:
        xs[0], ys[0] = on_ray
    return (0.1, 0.15, -0.05, xs, ys, ms)


@pytest.mark.parametrize("block", [1, 2, 4])
@pytest.mark.parametrize("dx,dy", [(0.01, 0.01), (0.02, 0.01), (0.05, 0.01), (0.2, 0.01), (0.01, 0.02), (0.01, 0.05),
                                   (0.01, 0.2)])
def test_tile_shapes(torch, block, dx, dy):
    """Every tile shape, with the last tiles cut by 1 to 63 rays, a ray on a
    star, and a window cutting through the rays."""
    for nx, ny, i0, j0 in ((257, 193, 0, 0), (16, 300, 7, 3), (321, 15, 0, 11), (1, 1, 5, 5)):
        x0, y0 = -0.5 * nx * dx, -0.5 * ny * dy
        on = (float(x0 + ((i0 + nx // 2) + 0.5) * dx), float(y0 + ((j0 + ny // 3) + 0.5) * dy))
        lens = _lens(nx, 300, max(nx * dx, ny * dy), on)
        pix = (-0.37, -0.41, 0.7 / 50, 0.9 / 41, 50, 41)
        with R.Context(lens) as ctx:
            ctx.set_expansion_block(block)
            _check(torch, ctx, lens, (x0, y0, dx, dy, nx, ny, i0, j0), pix)


@pytest.mark.parametrize("block", [2, 4])
@pytest.mark.parametrize("nx,ny,dx,dy", [(4161, 4033, 1e-3, 1e-3), (2100, 8209, 2.3e-3, 1e-3)])
def test_four_tiles_a_workgroup(torch, block, nx, ny, dx, dy):
    """Lattices of more than 4096 tiles, ragged: rows of four tiles a
    workgroup, some of them outside the lattice."""
    x0, y0 = -0.5 * nx * dx, -0.5 * ny * dy
    lens = _lens(nx, 800, 4.0)
    with R.Context(lens) as ctx:
        ctx.set_expansion_block(block)
        _check(torch, ctx, lens, (x0, y0, dx, dy, nx, ny, 0, 0), (-1.3, -1.1, 2.5 / 300, 2.1 / 280, 300, 280), 3000)


@pytest.mark.parametrize("block", [1, 2, 4])
@pytest.mark.parametrize("cluster", [200, 256, 300, 1500, 3000])
def test_near_lists(torch, block, cluster):
    """Clusters whose stars fit a tile's list, overflow it, and overflow the
    block's lists."""
    lens = _lens(cluster, 60, 6.0, (0.005, 0.005), cluster)
    with R.Context(lens) as ctx:
        ctx.set_expansion_block(block)
        _check(torch, ctx, lens, (-1.0, -1.0, 0.01, 0.01, 200, 200, 0, 0), (-1.0, -0.9, 0.02, 0.03, 90, 60))


@pytest.mark.parametrize("pix", [
    (-0.8, -0.7, 0.1, 0.1, 16, 14),                    # beta on pixel edges, P not a binary fraction
    (-1.0, -1.0, 1 / 3, 0.7, 6, 3),
    (-0.8, -0.7, 1e-3, 3e-3, 1600, 467),               # counts spread beyond the LDS window
    (0.0, -0.7, 0.1, 0.1, 8, 14),                      # X0 = 0: the division
    (-0.8, 1e-200, 0.1, 0.1, 16, 8),                   # |Y0| below the fast form's range
    (-1e-100, -0.8, 0.1, 0.05, 9, 31),                 # a tiny origin within it
    (-0.8, -0.7, 2.0 ** -301, 0.1, 4, 14),             # P below its range
    (-0.8, -0.7, 2.0 ** -300, 2.0 ** 300, 4, 1),       # the ends of its range
    (50.0, 50.0, 0.1, 0.1, 7, 7)])                     # no ray
def test_pixel_step(torch, pix):
    """beta = theta for an empty lens: rays on a grid of twentieths fall on
    the edges of tenths' pixels, where a quotient off by one unit in the last
    place changes the pixel."""
    lens = (0.0, 0.0, 0.0, np.zeros(0), np.zeros(0), np.zeros(0))
    with R.Context(lens) as ctx:
        for rays in ((-1.025, -1.025, 0.05, 0.05, 82, 82, 0, 0), (-1.0003, -0.9, 0.0031, 0.0083, 650, 220, 0, 0)):
            _check(torch, ctx, lens, rays, pix)


@pytest.mark.parametrize("spread", [1.0, 30.0])
@pytest.mark.parametrize("block", [1, 4])
@pytest.mark.parametrize("theta", [0.3, 0.25, 0.05])
def test_series_cut_by_distance(torch, block, theta, spread):
    """Star cells and their stars at distances from the opening radius to a
    hundred block radii: series of few to all terms, in the same waves."""
    rng = np.random.default_rng(int(100 * theta) + block)
    n = 4000
    r, phi = 0.3 * (spread * 400) ** rng.random(n), 2 * np.pi * rng.random(n)   # equally many per octave
    lens = (0.1, 0.15, -0.05, r * np.cos(phi), r * np.sin(phi), rng.uniform(1e-3, 2e-3, n))
    with R.Context(lens) as ctx:
        ctx.set_expansion(theta)
        ctx.set_expansion_block(block)
        ctx.set_expansion_cells("always")
        _check(torch, ctx, lens, (-0.8, -0.7, 0.008, 0.007, 200, 201, 0, 0), (-0.9, -0.8, 0.03, 0.02, 60, 81))
