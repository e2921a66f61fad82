"""Tensor-product cell operator (cell_tp.hip) against the oracle's dense cell
sums: every element order, widths around the work-group's units, a box with
three different cell sizes, and the form without workspace (cell colours)."""
import numpy as np
import pytest

from oracle import fe
from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


def plain(p, ncell, hi):
    w = dict(wl.PSP, lo=(0.0, -1.0, 2.0), hi=hi, ncell=ncell, p=p, nq=p + 1,
             xyz=np.zeros((1, 3)) + 1.0, enr_lmax=-1, Zs=np.ones(1))
    w["kb_D"] = 0.0
    return w


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("cols", [1, 7, 17, 65, 160, 203])
def test_cell_operator(p, cols):
    import torch
    from paper_2607_06848_amd import efe
    w = plain(p, (3, 2, 4), (4.0, 2.5, 9.0))
    mesh = fe.Mesh(w["lo"], w["hi"], w["ncell"], p, w["nq"])
    rng = np.random.default_rng([p, cols])
    vq = rng.normal(0.0, 2.0, (mesh.n_cells, mesh.nqp))
    inner = (1 - mesh.boundary)[:, None]
    X = rng.uniform(-1.0, 1.0, (mesh.n_nodes, cols)) * inner
    ref = mesh.cfe_apply(vq, X) * inner
    ctx = efe.Context(w)
    ctx.set_potential(torch.from_numpy(vq.ravel()).cuda())
    Y = ctx.apply_H(torch.from_numpy(X).cuda()).cpu().numpy()
    ctx.close()
    # 9 contractions of length <= 7 and 8 cells a node, each rounding once, on
    # values up to the sum of the magnitudes: well under 100 roundings
    scale = np.abs(ref).max()
    assert np.abs(Y - ref).max() < 100 * 2.0 ** -53 * 8 * scale


def test_without_room_for_cell_products():
    """A fixed scratch region that holds the blocks but not the cells' products:
    the operator is added colour by colour, to the same result."""
    import torch
    from paper_2607_06848_amd import efe
    w = plain(6, (8, 8, 8), (16.0, 15.0, 18.0))
    ctx = efe.Context(w)
    g = torch.Generator(device="cuda").manual_seed(3)
    vq = torch.rand(ctx.n_qpts, dtype=torch.float64, device="cuda", generator=g) - 1.0
    ctx.set_potential(vq)
    cols = 13
    # the blocks take 62 of 64 MiB; the products would take another 17
    assert 4 * ctx.rows * cols * 8 + ctx.rows * (cols + 1) * 8 < 64 << 20
    V = torch.rand(ctx.rows, cols, dtype=torch.float64, device="cuda", generator=g) - 0.5
    V[:ctx.n_nodes] *= torch.from_numpy(1.0 - ctx.tables()["boundary"]).cuda()[:, None]
    lam = torch.linspace(-1.0, 1.0, cols, dtype=torch.float64, device="cuda")
    A, B = V.clone(), V.clone()
    ctx.cheb_filter(A, lam, 6, 1.1, 600.0, -1.2)
    ctx.cheb_filter_noalloc(B, lam, 6, 1.1, 600.0, -1.2)
    err = float((A - B).abs().max() / A.abs().max())
    ctx.close()
    # six degrees, each within the bound of one apply
    assert err < 6 * 100 * 2.0 ** -53 * 8
