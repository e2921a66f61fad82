"""Poisson CG on the tensor-product stiffness (scf.hip): two SCF steps of a
small plain-CFE system for every element order, cells of three sizes and Gauss
rules with and without nq = p + 1, against the oracle's energies; and the
iteration limit."""
import numpy as np
import pytest

from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


def system(p, nq, ncell):
    w = dict(wl.PSP, lo=(0.0, 0.0, 0.0), hi=(10.0, 9.0, 11.0), ncell=ncell, p=p, nq=nq,
             xyz=np.array([[4.2, 4.4, 5.1], [6.3, 5.0, 6.2]]), enr_lmax=-1, Zs=np.full(2, 4.0))
    return w


@pytest.mark.parametrize("p,nq,ncell", [(1, 2, (9, 8, 10)), (2, 3, (5, 5, 6)), (3, 4, (4, 3, 5)),
                                        (3, 5, (4, 3, 5)), (4, 5, (3, 3, 4)), (5, 6, (3, 2, 3)),
                                        (6, 7, (2, 3, 2))])
def test_energies(p, nq, ncell):
    import torch
    from oracle import enrich, fe, scf
    from paper_2607_06848_amd import efe
    w = system(p, nq, ncell)
    mesh = fe.Mesh(w["lo"], w["hi"], w["ncell"], p, nq)
    s = enrich.EFESystem(mesh, w)
    es = scf.Electrostatics(mesh, w["xyz"], w["Zs"], w)
    V0, v0 = wl.random_block(s.rows, 8, 5), wl.random_vector(s.rows, 7)
    kT = 500 * scf.KB_HA_PER_K
    hist, _ = scf.scf(s, es, V0, v0, 8, 12, 8.0, kT, tol=1e-14, max_iter=2)
    ctx = efe.Context(w)
    V = torch.from_numpy(V0).cuda()
    lam = torch.zeros(8, dtype=torch.float64, device="cuda")
    for h in hist:
        r = ctx.scf_step(V, lam, torch.from_numpy(v0).cuda(), 12, passes_first=4, passes=1, kT=kT,
                         mix_beta=0.3, mix_history=8, cg_rtol=1e-12)
        # the bound of the SCF parity tests
        assert abs(r["E"] - h["E"]) < 1e-8 and abs(r["E_el"] - h["E_el"]) < 1e-8
    if hist:
        with pytest.raises(efe.EFEError) as e:
            ctx.scf_step(V, lam, torch.from_numpy(v0).cuda(), 12, kT=kT, cg_maxit=3)
        assert e.value.status == -4
    ctx.close()
