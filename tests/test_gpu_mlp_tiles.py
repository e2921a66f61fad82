"""Density-network kernels at the edges of their 64-point tiles and where a
work-group goes round its tile loop (256 groups backward, 512 forward), against
the FP64 oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# a point's outputs are FP32 sums of up to 128 products: 128 eps = 1.5e-5 of the
# largest; a gradient sums n points more, whose errors add like sqrt(n) at most
@pytest.mark.parametrize("n", [15, 63, 65, 129, 16385, 16449, 33000])
def test_mlp_tiles(n):
    from oracle import learned as L
    from paper_2607_06848_amd import efe
    rng = np.random.default_rng(n)
    th = L.init_params(n)
    X = rng.normal(size=(n, 25)).astype(np.float32)
    dy = rng.normal(size=n).astype(np.float32)
    y_ref, cache = L.forward(th, X.astype(np.float64))
    g_ref = L.backward(th, X.astype(np.float64), cache, dy.astype(np.float64))
    print("mlp tiles", n, flush=True)
    P = torch.as_tensor(np.asarray(th), dtype=torch.float32, device="cuda")
    Xd, dyd = torch.as_tensor(X, device="cuda"), torch.as_tensor(dy, device="cuda")
    acts = torch.full((3 * n * 128,), float("nan"), dtype=torch.float32, device="cuda")
    y = efe.efe_mlp_forward(P, Xd, acts)
    assert torch.equal(y, efe.efe_mlp_forward(P, Xd))
    np.testing.assert_allclose(y.cpu().numpy(), y_ref, rtol=0, atol=2e-5 * (1 + np.abs(y_ref).max()))
    z = acts.view(3, n, 128).cpu().numpy()
    for k in range(3):
        np.testing.assert_allclose(z[k], cache[k], rtol=0, atol=2e-5 * (1 + np.abs(cache[k]).max()))
    g = efe.efe_mlp_backward(P, Xd, acts, dyd).cpu().numpy()
    off = np.cumsum([0] + [int(np.prod(s)) for s in L.SHAPES])
    for i in range(len(L.SHAPES)):
        a, b = g_ref[off[i]:off[i + 1]], g[off[i]:off[i + 1]]
        assert np.abs(a - b).max() < 1e-4 * (np.abs(a).max() + 1e-30), i
