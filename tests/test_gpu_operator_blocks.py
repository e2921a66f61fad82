"""Operators of a potential at the edges of their work split (setup.hip, couple.hip):
16, 17 and 32 functions on a cell (H^E_ee formed beside E_c), 36 (over boxes), and
elements whose rows and steps leave remainders, against the oracle."""
import numpy as np
import pytest

from oracle import enrich, fe
from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,nq", [(2, 3), (3, 5), (4, 5)])
@pytest.mark.parametrize("natoms,lmax,functions", [(4, 1, 16), (17, 0, 17), (8, 1, 32), (4, 2, 36)])
def test_apply_H(p, nq, natoms, lmax, functions):
    import torch
    from paper_2607_06848_amd import efe
    rng = np.random.default_rng([p, natoms])
    w = dict(wl.PSP, lo=(0.0,) * 3, hi=(8.0, 9.0, 7.0), ncell=(4, 4, 3), p=p, nq=nq,
             xyz=rng.uniform(3.3, 4.2, (natoms, 3)), enr_lmax=lmax, enr_rcut=2.2, kb_rcut=2.5,
             Zs=np.full(natoms, 4.0))
    mesh = fe.Mesh(w["lo"], w["hi"], w["ncell"], p, nq)
    s = enrich.EFESystem(mesh, w)
    vq = rng.normal(0.0, 1.0, (mesh.n_cells, mesh.nqp))
    s.set_potential(vq)
    ctx = efe.Context(w)
    assert -(-functions // 16) * 16 == ctx.coupling()[1]
    ctx.set_potential(torch.from_numpy(vq.ravel()).cuda())
    mask = np.zeros(s.rows)
    mask[s.active()] = 1.0
    X = rng.uniform(-1.0, 1.0, (s.rows, 5)) * mask[:, None]
    ref = s.apply_H(X)
    for _ in range(2):                     # the second potential over the first's results
        Y = ctx.apply_H(torch.from_numpy(X).cuda()).cpu().numpy()
        # the parity bound of the H apply
        assert np.abs(Y - ref).max() < 1e-12 * np.abs(ref).max()
        ctx.set_potential(torch.from_numpy(vq.ravel()).cuda())
    ctx.close()
