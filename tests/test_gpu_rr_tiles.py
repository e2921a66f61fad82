"""Rayleigh-Ritz at the edges of its tiles (rr.hip: 16-column tiles, register
tiles of 1, 3, 6 and 10 of them, the pair and quad loads, 161 vectors on the
general path) with odd leading dimensions, against the oracle on the 2-atom
workload."""
import numpy as np
import pytest

from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pair():
    import torch
    from oracle import enrich, fe
    from paper_2607_06848_amd import efe
    w = wl.make("eig2")
    mesh = fe.Mesh(w["lo"], w["hi"], w["ncell"], w["p"], w["nq"])
    s = enrich.EFESystem(mesh, w)
    vq = np.random.default_rng(3).normal(0.0, 1.0, (mesh.n_cells, mesh.nqp))
    s.set_potential(vq)
    ctx = efe.Context(w)
    ctx.set_potential(torch.from_numpy(vq.ravel()).cuda())
    yield s, ctx
    ctx.close()


@pytest.mark.parametrize("n,pad", [(2, 0), (15, 1), (16, 0), (17, 3), (32, 0), (49, 0), (50, 2),
                                   (96, 0), (98, 1), (130, 0), (159, 1), (160, 2), (161, 0)])
def test_tiles(pair, n, pad):
    import torch
    from oracle import eigen
    s, ctx = pair
    mask = np.zeros(s.rows)
    mask[s.active()] = 1.0
    V0 = wl.random_block(s.rows, n, 31)      # boundary rows not zero: they come back zero
    Vr, lam, res = eigen.rayleigh_ritz(s.apply_H, s.apply_M, V0 * mask[:, None], mask)
    Vd = torch.zeros(s.rows, n + pad, dtype=torch.float64, device="cuda")
    Vd[:, :n] = torch.from_numpy(V0).cuda()
    W = Vd.clone()
    lg, rg = ctx.rayleigh_ritz(Vd[:, :n])
    l2, _ = ctx.rayleigh_ritz(W[:, :n], want_res=False)
    lg, rg, l2 = lg.cpu().numpy(), rg.cpu().numpy(), l2.cpu().numpy()
    Vg, Wg = Vd[:, :n].cpu().numpy(), W[:, :n].cpu().numpy()
    # the bounds of the other Rayleigh-Ritz parity tests
    assert np.abs(lg - lam).max() <= 1e-10 * max(1.0, np.abs(lam).max())
    assert np.abs(l2 - lam).max() <= 1e-10 * max(1.0, np.abs(lam).max())
    assert np.abs(rg - res).max() <= 1e-9 * max(1.0, res.max())
    for X in (Vg, Wg):
        assert np.abs(X.T @ s.apply_M(X) - np.eye(n)).max() < 1e-11
        assert not X[mask == 0.0].any()
    if pad:
        assert not Vd[:, n:].any()
