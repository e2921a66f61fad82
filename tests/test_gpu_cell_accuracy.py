"""Rounding of the tensor-product cell operator: no larger than that of the dense
cell products.  Under a constant potential the Gauss rules with p + 1 points
(tensor products) and p + 2 (dense cells) give the same operator, so both run on
the same nodal values, against the operator in extended precision.  (No rule has
the 8 points that p = 6 would take.)"""
import numpy as np
import pytest

from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu
LD = np.longdouble


def legendre(n, x):
    a, b = np.ones_like(x), x
    for k in range(1, n):
        a, b = b, ((2 * k + 1) * x * b - k * a) / LD(k + 1)
    return b, n * (x * b - a) / (x * x - 1)


def rules(p):
    """GLL nodes, and the 1-D mass and stiffness matrices of their basis on [-1, 1]."""
    x = -np.cos(np.pi * np.arange(1, p) / p).astype(LD)
    for _ in range(60):
        P, d = legendre(p, x)
        x = x - d / ((2 * x * d - p * (p + 1) * P) / (1 - x * x))
    xn = np.concatenate([[LD(-1)], x, [LD(1)]])
    q = -np.cos(np.pi * (np.arange(p + 1) + 0.75) / (p + 1.5)).astype(LD)
    for _ in range(60):
        P, d = legendre(p + 1, q)
        q = q - P / d
    w = 2 / ((1 - q * q) * legendre(p + 1, q)[1] ** 2)
    N, D = np.ones((p + 1, p + 1), LD), np.zeros((p + 1, p + 1), LD)
    for a in range(p + 1):
        others = [b for b in range(p + 1) if b != a]
        for b in others:
            N[:, a] *= (q - xn[b]) / (xn[a] - xn[b])
            t = 1 / (xn[a] - xn[b]) * np.ones_like(q)
            for c in others:
                if c != b:
                    t = t * (q - xn[c]) / (xn[a] - xn[c])
            D[:, a] += t
    return xn, (N.T * w) @ N, (D.T * w) @ D


def along(M, a, d):
    return np.moveaxis(np.tensordot(M, a, (1, d)), 0, d)


def exact(p, nc, h, M, K, v0, X):
    n = nc * p + 1
    Y = np.zeros((n, n, n, X.shape[-1]), LD)
    Xl = X.reshape(n, n, n, -1).astype(LD)          # z, y, x
    m, k = M * LD(h) / 2, K * 2 / LD(h)
    for c in np.ndindex(nc, nc, nc):
        s = tuple(slice(i * p, i * p + p + 1) for i in c)
        mm = [along(m, along(m, Xl[s], i), j) for i, j in ((1, 2), (0, 2), (0, 1))]
        Y[s] += LD(v0) * along(m, mm[0], 0) + sum(along(k, mm[d], d) for d in range(3)) / 2
    for d in range(3):
        np.moveaxis(Y, d, 0)[[0, -1]] = 0
    return Y.reshape(n ** 3, -1)


@pytest.mark.parametrize("p", [1, 2, 3, 4, 5])
def test_rounding_against_dense_cells(p):
    import torch
    from paper_2607_06848_amd import efe
    nc, L, cols = (6 if p < 4 else 4), 8.0, 8
    h, v0 = L / nc, -0.75
    xn, M, K = rules(p)
    ax = np.concatenate([(xn[:-1] + 1) / 2 * h + c * h for c in range(nc)] + [[L]]).astype(float)
    z, y, x = np.meshgrid(ax, ax, ax, indexing="ij")
    rng = np.random.default_rng(p)
    smooth = [np.exp(-rng.uniform(0.15, 0.6) * ((x - 4 - rng.normal(0, 0.4)) ** 2 + (y - 4) ** 2
                                                + (z - 4) ** 2))
              * (1 + rng.normal() * (x - 4) + rng.normal() * (z - 4) * (y - 4)) for _ in range(cols)]
    inner = np.ones_like(x)
    for d in range(3):
        np.moveaxis(inner, d, 0)[[0, -1]] = 0
    fields = {"smooth": np.stack(smooth, -1), "random": rng.uniform(-1, 1, x.shape + (cols,))}
    for kind, X in fields.items():
        X = (X * inner[..., None]).reshape(-1, cols)
        ref = exact(p, nc, h, M, K, v0, X)
        err = []
        for nq in (p + 1, p + 2):
            w = dict(wl.PSP, lo=(0.0,) * 3, hi=(L,) * 3, ncell=(nc,) * 3, p=p, nq=nq,
                     xyz=np.zeros((1, 3)) + 4.0, enr_lmax=-1, Zs=np.ones(1))
            w["kb_D"] = 0.0
            ctx = efe.Context(w)
            ctx.set_potential(torch.full((ctx.n_qpts,), v0, dtype=torch.float64, device="cuda"))
            Y = ctx.apply_H(torch.from_numpy(X).cuda()).cpu().numpy()
            ctx.close()
            err.append(float((np.abs(Y - ref).max(0) / np.abs(ref).max(0)).mean()))
        print(p, kind, err, flush=True)
        # the mean over the columns of the largest error: no larger than dense
        assert err[0] <= err[1], (kind, err)
