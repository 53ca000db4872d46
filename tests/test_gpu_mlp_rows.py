"""The network's one-launch row kernel and its gradient kernel at the edges of
their tiles, and the layer-by-layer path beyond the row kernel's sizes,
against the FP64 oracle."""
import numpy as np
import pytest

from oracle import surrogate as OS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("needs a GPU")
    return t


# 64 columns a wave, 16 steps a block, 4, 8 or 16 rows a workgroup (above 2048
# and 4096 rows), 16 x 16 gradient tiles; layers of at most 512, then the
# layer-by-layer path
@pytest.mark.parametrize("n_in,h,n_out,B", [
    (1, 1, 1, 1), (4, 64, 64, 4), (4, 65, 63, 5), (16, 16, 16, 3), (17, 127, 129, 33), (4, 256, 64, 2049),
    (5, 96, 20, 4097), (512, 512, 512, 7), (3, 512, 500, 4097), (4, 513, 64, 45), (513, 32, 9, 12)])
def test_network_at_tile_edges_matches_oracle(torch, n_in, h, n_out, B):
    """The tolerances are those of the other network tests: FP32 sums of at
    most 513 terms (relative error of a term below 513 x 2^-24 = 3.1e-5)
    behind GELUs and a softmax."""
    from paper_1703_09707_amd import surrogate as S
    rng = np.random.default_rng(n_in * 7919 + h * 31 + n_out + B)
    params = OS.init_params(n_in, h, n_out, rng)
    params = (params + rng.normal(0, 0.05, params.shape)).astype(np.float32)
    x = rng.standard_normal((B, n_in)).astype(np.float32)
    t = rng.random((B, n_out)).astype(np.float32)
    t /= t.sum(axis=1, keepdims=True)
    net = S.MLP(params, n_in=n_in, n_hidden=h, n_out=n_out, max_batch=B)
    try:
        xg, tg = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
        want, _ = OS.forward(params, x, n_in, h, n_out)
        np.testing.assert_allclose(net.forward(xg).cpu().numpy(), want, rtol=2e-4, atol=1e-7)
        g, loss = net.gradient(xg, tg)
        gw = OS.gradients(params, x, t, n_in, h, n_out)
        assert abs(loss.item() - OS.loss(params, x, t, n_in, h, n_out)) < 1e-5
        # one output: p = t = 1, the gradient is zero up to rounding
        assert np.linalg.norm(g.cpu().numpy() - gw) <= 1e-4 * np.linalg.norm(gw) + 1e-7
        net.adam_step(1e-3)   # both BF16 layouts follow the masters
        p2, _, _ = OS.adam(params, g.cpu().numpy(), np.zeros_like(params), np.zeros_like(params), 1, 1e-3)
        np.testing.assert_allclose(net.params(), p2, rtol=1e-6, atol=1e-7)
        got = net.params()
        want, _ = OS.forward(got, x, n_in, h, n_out)
        np.testing.assert_allclose(net.forward(xg).cpu().numpy(), want, rtol=2e-4, atol=1e-7)
        g2, _ = net.gradient(xg, tg)
        gw = OS.gradients(got, x, t, n_in, h, n_out)
        assert np.linalg.norm(g2.cpu().numpy() - gw) <= 1e-4 * np.linalg.norm(gw) + 1e-7
    finally:
        net.close()
