"""Light curves beyond the threads of one launch (2^32): the curves of a few
thousand tracks repeat over all the launches."""
import pytest

from paper_1703_09707_amd import raysh as R

pytestmark = pytest.mark.gpu


# the kernel of a wave a chunk, from 64 samples on (2^33 threads), and the one
# of four samples a thread (two launches of 2^31 threads)
@pytest.mark.parametrize("n_tracks,n_samples", [((1 << 27) + 700, 64), ((1 << 29) + 333, 17)])
def test_more_than_one_launch(n_tracks, n_samples):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU")
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (8 * n_samples + 44) * n_tracks + (8 << 30):
        pytest.skip("not enough free device memory")
    g = torch.Generator().manual_seed(n_samples)
    mu = torch.rand((40, 50), generator=g, dtype=torch.float64).cuda()
    grid = (0.0, 0.0, 1.0, 1.0, 50, 40)
    k = 4096
    few = [(torch.rand(k, generator=g, dtype=torch.float64) * (side - 2) + 1).cuda() for side in (50, 40, 50, 40)]
    want = R.light_curves(mu, grid, *few, n_samples)
    many = [t.repeat(-(-n_tracks // k))[:n_tracks].contiguous() for t in few]
    got = R.light_curves(mu, grid, *many, n_samples)
    whole = n_tracks // k * k
    for part in got[:whole].view(-1, k, n_samples).split(1024):
        assert bool((part == want).all())
    assert torch.equal(got[whole:], want[:n_tracks - whole])
    del got, many
    torch.cuda.empty_cache()
