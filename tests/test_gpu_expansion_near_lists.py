"""Tiles with more near stars than fit their own list (256) take the same
terms as others: their near stars directly, the block's other near stars in
their polynomial."""
import numpy as np
import pytest

from oracle import shooter as ora
from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu

PIX = (-0.9, -0.8, 0.03, 0.04, 60, 40)
BETA_TOL = 1e-12   # of the error scale S: the FP64 bar of the other expansion tests


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    return t


def _ring(rng, n, lo, hi):
    r, phi = rng.uniform(lo, hi, n), 2 * np.pi * rng.random(n)
    return r * np.cos(phi), r * np.sin(phi)


@pytest.mark.parametrize("block", [1, 2, 4])
@pytest.mark.parametrize("massless", [100, 216, 217, 300, 700, 1500])
def test_long_lists_take_the_same_terms(torch, block, massless):
    """128 x 128 rays (tile radius 0.445, block radius 0.898: opened within
    1.78 and 3.59), 40 near stars, 200 far from the tiles but near the 2 x 2
    block, and massless stars, which change no sum: those near all tiles or
    those far from them leave every ray's beta the same bit for bit."""
    rng = np.random.default_rng(massless)
    d = 0.01
    x, y = (np.concatenate(v) for v in zip(_ring(rng, 40, 0.0, 1.0), _ring(rng, 200, 2.3, 3.4)))
    m = rng.uniform(1e-3, 2e-3, x.size)
    order = rng.permutation(x.size + massless)
    betas = []
    for lo, hi in ((0.0, 0.3), (3.2, 3.4)):
        zx, zy = _ring(rng, massless, lo, hi)
        lens = (0.1, 0.15, -0.05, np.concatenate([x, zx])[order], np.concatenate([y, zy])[order],
                np.concatenate([m, np.zeros(massless)])[order])
        rays = (-64 * d, -64 * d, d, d, 128, 128, 0, 0)
        with R.Context(lens) as ctx:
            ctx.set_expansion_block(block)
            betas.append([t.cpu().numpy() for t in ctx.shoot(rays, "fp64_expansion", PIX)])
    ox, oy, _ = ora.shoot(lens, rays, PIX)
    s = ora.error_scale_block(lens, rays)
    for (near, far, want) in zip(betas[0][:2], betas[1][:2], (ox, oy)):
        assert np.all(np.abs(near - want) <= BETA_TOL * s)
        np.testing.assert_array_equal(near, far)
