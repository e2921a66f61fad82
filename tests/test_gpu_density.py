"""Output density of one SCF step from the vectors the step returns, against the
oracle's density of the same vectors: every element order of the 1-D
contractions, a Gauss rule without them, ragged column counts, no to several
enriched atoms a cell, and more than one 160-column chunk."""
import numpy as np
import pytest

from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,nq,lmax,natoms,nvec", [(1, 2, 1, 2, 7), (2, 3, 2, 3, 17), (3, 4, 0, 2, 16),
                                                   (4, 5, 2, 4, 33), (5, 6, 1, 2, 21), (6, 7, 2, 3, 40),
                                                   (4, 6, 2, 2, 18), (3, 4, 2, 3, 170),
                                                   (4, 5, -1, 2, 12)])
def test_density(p, nq, lmax, natoms, nvec):
    import torch
    from oracle import enrich, fe, scf
    from paper_2607_06848_amd import efe
    rng = np.random.default_rng([p, nq, natoms, nvec])
    n = 4 if p > 1 else 7
    w = dict(wl.PSP, lo=(0.0,) * 3, hi=(9.0,) * 3, ncell=(n,) * 3, p=p, nq=nq, enr_lmax=lmax,
             xyz=wl.jittered_lattice(2, 3.0, 0.1, p)[:natoms] + 3.0, enr_rcut=2.5, kb_rcut=3.0,
             Zs=np.full(natoms, 2.0))
    mesh = fe.Mesh(w["lo"], w["hi"], w["ncell"], p, nq)
    s = enrich.EFESystem(mesh, w)
    print("density", p, nq, lmax, natoms, nvec, s.rows, flush=True)
    ctx = efe.Context(w)
    V = torch.from_numpy(wl.random_block(s.rows, nvec, 5)).cuda()
    lam = torch.zeros(nvec, dtype=torch.float64, device="cuda")
    kT = 0.1     # every column occupied to some extent
    ctx.scf_step(V, lam, torch.from_numpy(wl.random_vector(s.rows, 7)).cuda(), 6, passes_first=1,
                 passes=1, kT=kT, mix_beta=0.3, mix_history=4, cg_rtol=1e-8)
    _, f = scf.fermi_level(lam.cpu().numpy(), 2.0 * natoms, kT)
    ref = scf.density(s, V.cpu().numpy(), f)
    rho = ctx.get_density(1).cpu().numpy().reshape(ref.shape)
    # sums of a few hundred FP64 terms a value; f to 1e-14 / kT of the bisection
    assert np.abs(rho - ref).max() < 1e-11 * np.abs(ref).max()
    ctx.close()
