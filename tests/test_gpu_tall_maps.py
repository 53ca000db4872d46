"""Maps of few columns and 2^26 rows: the passes with a wave per row would need
a grid of 2^32 threads, so a thread per output serves these maps.  The rows
repeat every 64, and so must the results, which a short map gives too."""
import pytest

from paper_1703_09707_amd import raysh as R
from paper_1703_09707_amd import surrogate

pytestmark = pytest.mark.gpu

NX, NY = 6, 1 << 26
PX, PY = 1.0, 0.031


@pytest.fixture(scope="module")
def maps():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    g = torch.Generator().manual_seed(3)
    one = torch.randint(0, 90, (64, NX), generator=g, dtype=torch.int32).cuda()
    return one.repeat(NY // 64, 1), one.repeat(8, 1)


# radii (1, 32), and a disk's (2, 80): both through their sliding or prefix form on maps less tall
@pytest.mark.parametrize("profile,size,ry", [("gaussian", 0.33, 32), ("disk", 2.5, 80)])
def test_source_map(maps, profile, size, ry):
    import torch
    tall, short = maps
    want, _ = R.source_map(short, (0.0, 0.0, PX, PY, NX, 512), 0.3, profile, size)
    mu, grid = R.source_map(tall, (0.0, 0.0, PX, PY, NX, NY), 0.3, profile, size)
    assert mu.shape == (NY - 2 * ry, grid[4])
    whole = mu.shape[0] // 64 * 64
    assert bool((mu[:whole].view(-1, 64, grid[4]) == want[:64]).all())
    assert torch.equal(mu[whole:], want[:mu.shape[0] - whole])


def test_histogram(maps):
    tall, short = maps
    sigma, ry = 0.33, 32
    args = (0.3, sigma, PX, PY, 2.0)
    b, h = surrogate.Histogrammer(NX, 512)(short, *args)
    bt, ht = surrogate.Histogrammer(NX, NY)(tall, *args)
    per, rows = b.long() * 64, 512 - 2 * ry
    assert bool((per % rows == 0).all())   # the short map's rows are whole periods
    assert bool((bt.long() == per // rows * ((NY - 2 * ry) // 64)).all())
    assert bool(((ht - h).abs() <= 2.0 ** -23 * h).all())
