"""Which form a one-pass FP64 launch runs in: the shape that raysh_set_tile or
the tuner has set, else the lattice's own (waves that share a tile where the
context's shape would leave compute units idle)."""
import numpy as np
import pytest

from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu

PIX = (-0.9, -0.8, 1.7 / 45, 1.9 / 52, 45, 52)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _rays(nx, ny):
    return (-1.25, -1.25, 2.5 / nx, 2.5 / nx, nx, ny, 0, 0)


def _lens(n, seed=0):
    rng = np.random.default_rng(n + seed)
    return (0.1, 0.1, -0.05, rng.uniform(-3, 3, n), rng.uniform(-3, 3, n), rng.uniform(0.01, 0.05, n))


def _shoot(ctx, rays):
    return [t.cpu().numpy() for t in ctx.shoot(rays, "fp64", PIX)]


def _same(a, b):
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


def _set(ctx, t):
    ctx.set_tile("fp64", t[0], t[1], share=t[2], star_tile=t[3])


@pytest.mark.parametrize("nx,ny", [(500, 490), (100, 100)])
def test_tuned_shape_runs(torch, tmp_path, nx, ny):
    """After raysh_autotune, and after a hit of its cache, the shape it returns
    is the one that runs, on a lattice whose own form would be another."""
    rays, lens = _rays(nx, ny), _lens(300)
    cache = str(tmp_path / "cache")
    for _ in ("timed", "cached"):
        with R.Context(lens) as ctx, R.Context(lens) as fixed:
            t = ctx.autotune(rays, PIX, "fp64", cache_path=cache)
            _set(fixed, t)
            _same(_shoot(ctx, rays), _shoot(fixed, rays))


def test_batch_tuned_shape_runs(torch):
    rays = [_rays(300, 200), _rays(120, 500)]
    lenses = [_lens(200, 1), _lens(150, 2)]
    ctxs = [R.Context(l) for l in lenses]
    try:
        t = R.autotune_batch(ctxs, rays, [PIX, PIX], "fp64")
        for ctx, lens, r in zip(ctxs, lenses, rays):
            with R.Context(lens) as fixed:
                _set(fixed, t)
                _same(_shoot(ctx, r), _shoot(fixed, r))
    finally:
        for c in ctxs:
            c.close()


def test_wide_lattice_of_few_rows(torch):
    """2^27 columns: the form with 1024 threads for 32 x 16 rays would need
    2^32 threads.  The map equals that of a set shape."""
    nx = (1 << 27) + 77
    rays = (-1.25, -0.3, 2.5 / nx, 0.3, nx, 2, 0, 0)
    pix = (-2.0, -2.0, 0.05, 0.05, 80, 80)
    with R.Context(_lens(150)) as ctx:
        m, n = ctx.map(rays, pix, "fp64", n_binned=True)
        _set(ctx, (8, 4, 16, 1))
        w, nw = ctx.map(rays, pix, "fp64", n_binned=True)
    # rays within a rounding of a pixel's edge (1e-14 of its 0.05) may go either way
    assert abs(int(n) - int(nw)) <= 10
    assert int((m - w).abs().sum()) <= 20
    assert int(n) == int(m.sum(dtype=torch.int64)) > nx // 2


@pytest.mark.parametrize("shape", [(8, 4, 16, 1), (2, 2, 2, 2), (4, 4, 8, 4)])
def test_set_shape_is_exact(torch, shape):
    """In a set shape a ray's beta is the whole lattice's, bit for bit, in every
    block that begins at a whole tile, and a batch's maps are the single
    launches'."""
    nx, ny = 700, 650
    rays, lens = _rays(nx, ny), _lens(230)
    with R.Context(lens) as ctx:
        _set(ctx, shape)
        whole = _shoot(ctx, rays)
        tw, th = 16 * shape[0], 16 * shape[1]
        for i0, j0, w, h in ((0, 0, nx, 2 * th), (0, 3 * th, nx, 101), (2 * tw, th, 300, ny - th), (tw, 0, 33, 7)):
            part = _shoot(ctx, rays[:4] + (w, h, i0, j0))
            for a, b in zip(whole, part):
                np.testing.assert_array_equal(a[j0:j0 + h, i0:i0 + w], b)
        others = [_rays(300, 200), rays, _rays(90, 1000)]
        single = [ctx.map(r, PIX, "fp64") for r in others]
        batch = R.map_batch([ctx] * 3, others, [PIX] * 3, "fp64")
        assert all(torch.equal(a, b) for a, b in zip(single, batch))


def test_full_lattice_is_exact_by_default(torch):
    """A lattice that fills the device: the batch's map and the sum of its
    bands' (each of them full too) are the single launch's, with no shape set."""
    nx = 4096
    rays, lens = _rays(nx, 2 * nx), _lens(60)
    with R.Context(lens) as ctx:
        whole = ctx.map(rays, PIX, "fp64")
        assert torch.equal(R.map_batch([ctx], [rays], [PIX], "fp64")[0], whole)
        acc = torch.zeros_like(whole)
        for j0 in (0, nx):
            ctx.map(rays[:5] + (nx, 0, j0), PIX, "fp64", counts=acc)
        assert torch.equal(acc, whole)
        beta = ctx.shoot(rays, "fp64", PIX)
        for j0 in (0, nx):
            part = ctx.shoot(rays[:5] + (nx, 0, j0), "fp64", PIX)
            assert all(torch.equal(a[j0:j0 + nx], b) for a, b in zip(beta, part))


@pytest.mark.parametrize("precision,shape,nx", [("fp64", (2, 2, 2, 2), (1 << 29) + 3200),
                                                ("fp32_bulk", (4, 4, 0, 128), (1 << 30) + 6400)])
def test_grid_beyond_a_launch_is_refused(torch, precision, shape, nx):
    """Tiles of 256 threads for a row of nx rays: 2^32 threads and some, which HIP
    launches without an error and leaves undone."""
    rays = (-1.25, -0.3, 2.5 / nx, 0.3, nx, 1, 0, 0)
    with R.Context(_lens(2)) as ctx:
        ctx.set_tile(precision, shape[0], shape[1], share=shape[2], star_tile=shape[3])
        counts = torch.zeros((PIX[5], PIX[4]), dtype=torch.int32, device="cuda")
        with pytest.raises(R.RayshError):
            ctx.map(rays, PIX, precision, counts=counts)
        assert int(counts.sum()) == 0
