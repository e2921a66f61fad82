"""Projector coefficients over enough blocks for the chunked gather (more than 2,048
16-row blocks times 16-column parts), in the list of their own that FP32 applies and
plain systems have, against the same columns in the variant for few."""
import numpy as np
import pytest

from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


def projector_blocks(ctx, w):
    """16-row blocks of P^C over the boxes of 8 x 8 x 8 nodes."""
    ptr, cells = ctx.support(1)
    nc, p = w["ncell"], w["p"]
    count = {}
    for i in range(ctx.natoms):
        boxes = set()
        for c in cells[ptr[i]:ptr[i + 1]]:
            ijk = c % nc[0], c // nc[0] % nc[1], c // (nc[0] * nc[1])
            r = [range(max(k * p, 1) // 8, min(k * p + p, n * p - 1) // 8 + 1)
                 for k, n in zip(ijk, nc)]
            boxes |= {(x, y, z) for x in r[0] for y in r[1] for z in r[2]}
        for b in boxes:
            count[b] = count.get(b, 0) + 1
    return sum(-(-n // 16) for n in count.values())


@pytest.mark.parametrize("lmax", [-1, 0])
def test_wide_and_narrow(lmax):
    import torch
    from paper_2607_06848_amd import efe
    rng = np.random.default_rng(3)
    xyz = rng.uniform(2.5, 7.5, (27, 3))
    w = dict(wl.PSP, lo=(0.0,) * 3, hi=(10.0,) * 3, ncell=(24,) * 3, p=2, nq=3, xyz=xyz,
             enr_lmax=lmax, enr_rcut=1.5, kb_rcut=4.0, Zs=np.full(27, 4.0))
    ctx = efe.Context(w)
    n = projector_blocks(ctx, w)
    assert n <= 2048 < 10 * n
    ctx.set_potential(ctx.local_potential(), 1 << efe.EFE_FP32)
    g = torch.Generator(device="cuda").manual_seed(1)
    X = torch.rand(ctx.rows, 160, dtype=torch.float64, device="cuda", generator=g) - 0.5
    X[:ctx.n_nodes] *= torch.from_numpy(1.0 - ctx.tables()["boundary"]).cuda()[:, None]
    # sums of about 1e4 terms of either sign, each rounding once; FP32: the coupling
    # of the coupling tests
    for prec, tol in ((efe.EFE_FP64, 1e-12), (efe.EFE_FP32, 1e-12 if lmax < 0 else 1e-5)):
        Y = ctx.apply_H_prec(X, prec)
        scale = float(Y.abs().max())
        for j in (0, 37, 152):
            y = ctx.apply_H_prec(X[:, j:j + 8].contiguous(), prec)
            assert float((Y[:, j:j + 8] - y).abs().max()) < tol * scale
    ref = ctx.apply_H(X)
    assert float((Y - ref).abs().max()) < (1e-12 if lmax < 0 else 1e-5) * float(ref.abs().max())
    ctx.close()
