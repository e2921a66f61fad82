"""An atom whose enrichment reaches no cell of the mesh: no operator of the
coupling exists, and the applies are those of the mesh alone (the plain
system's) with zero rows for the enrichment functions.

Both contexts run the same cell kernel on the same tables.  Only the way of
the cells' products to the nodes may differ, at most 8 products a node, so a
row agrees to 8 roundings of its largest product, 8 * 2^-53 < 1e-15 times the
largest entry of the field's products; 1e-13 of the result's largest entry
leaves two digits for their cancellation."""
import numpy as np
import pytest
import torch

from paper_2607_06848_amd import efe
from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,nq", [(3, 4), (2, 4)])
@pytest.mark.parametrize("ncols", [1, 17])
def test_atom_outside_the_mesh(p, nq, ncols):
    w = dict(wl.PSP, lo=(0.0, 0.0, 0.0), hi=(6.0, 5.0, 7.0), ncell=(2, 3, 2), p=p, nq=nq,
             xyz=np.full((1, 3), -20.0), Zs=np.full(1, 4.0), enr_lmax=1, enr_rcut=3.0, kb_D=0.0)
    far, plain = efe.Context(w), efe.Context(dict(w, enr_lmax=-1))
    rng = np.random.default_rng(5)
    vq = torch.from_numpy(rng.normal(0.0, 1.0, far.n_qpts)).cuda()
    X = rng.uniform(-1.0, 1.0, (far.rows, ncols))
    X[:far.n_nodes] *= (1.0 - far.tables()["boundary"])[:, None]
    assert far.rows == far.n_nodes + 4 and plain.rows == plain.n_nodes == far.n_nodes
    for c in (far, plain):
        c.set_potential(vq)
    Y = far.apply_H(torch.from_numpy(X).cuda()).cpu().numpy()
    R = plain.apply_H(torch.from_numpy(X[:far.n_nodes].copy()).cuda()).cpu().numpy()
    assert np.abs(Y[:far.n_nodes] - R).max() <= 1e-13 * np.abs(R).max()
    assert not Y[far.n_nodes:].any()
    far.close()
    plain.close()
