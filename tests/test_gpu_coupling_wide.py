"""Coupling blocks on a mesh with enough boxes and bricks for the chunked
kernels (512 boxes' items, 1,024 bricks), where the small meshes of the other
tests take the variants for few work-groups: every column tile against the
oracle, and the few columns that the two variants share."""
import numpy as np
import pytest

from oracle import enrich, fe
from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_apply_H_many_boxes():
    import torch
    from paper_2607_06848_amd import efe
    # 43^3 nodes: 216 boxes, 1,331 bricks; 16 atoms over nearly all of them: up
    # to ten 16-row blocks, three work items a box
    rng = np.random.default_rng(7)
    xyz = rng.uniform(3.5, 6.5, (16, 3))
    w = dict(wl.PSP, lo=(0.0,) * 3, hi=(10.0,) * 3, ncell=(14, 14, 14), p=3, nq=4, xyz=xyz,
             enr_lmax=2, enr_rcut=5.0, kb_rcut=5.5, Zs=np.full(len(xyz), 4.0))
    mesh = fe.Mesh(w["lo"], w["hi"], w["ncell"], 3, 4)
    s = enrich.EFESystem(mesh, w)
    vq = rng.normal(0.0, 1.0, (mesh.n_cells, mesh.nqp))
    s.set_potential(vq)
    ctx = efe.Context(w)
    ctx.set_potential(torch.from_numpy(vq.ravel()).cuda(), 1 << efe.EFE_FP32)
    mask = np.zeros(s.rows)
    mask[s.active()] = 1.0
    X = rng.uniform(-1.0, 1.0, (s.rows, 160)) * mask[:, None]
    ref = s.apply_H(X)
    for cols in (1, 3, 16, 17, 37, 64, 66, 97, 129, 160):
        for ld in (cols, cols + 3):
            Xd = torch.zeros(s.rows, ld, dtype=torch.float64, device="cuda")
            Xd[:, :cols] = torch.from_numpy(X[:, :cols]).cuda()
            for prec, tol in ((efe.EFE_FP64, 1e-12), (efe.EFE_FP32, 1e-5)):
                Y = ctx.apply_H_prec(Xd[:, :cols], prec).cpu().numpy()
                # the parity bound of the H apply; FP32: 2^-24 times the
                # cancellation between B and C H
                assert np.abs(Y - ref[:, :cols]).max() < tol * np.abs(ref).max(), (cols, ld, prec)
    ctx.close()
