"""A density that is not a number at some Gauss points: the Poisson solve for it
runs no iteration and the step goes on with the potential of before, which the
next step starts from."""
import math

import pytest

from paper_2607_06848_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_step_after_a_density_of_nan():
    import torch
    from paper_2607_06848_amd import efe
    w = wl.make("eig2")

    def step(ctx, rho):
        V = torch.from_numpy(wl.random_block(ctx.rows, 12, 5)).cuda()
        lam = torch.zeros(12, dtype=torch.float64, device="cuda")
        v0 = torch.from_numpy(wl.random_vector(ctx.rows, 7)).cuda()
        ctx.set_density(rho)
        return ctx.scf_step(V, lam, v0, 10, passes_first=2)

    ctx = efe.Context(w)
    rho = ctx.get_density(2)
    zero = step(ctx, rho)                  # no source: phi = 0
    ctx.close()
    ctx = efe.Context(w)
    ref = step(ctx, 0.9 * rho)
    ctx.close()
    ctx = efe.Context(w)
    bad = rho.clone()
    bad[17] = float("nan")
    r = step(ctx, bad)
    # the bound of the SCF parity tests
    assert math.isnan(r["drho"]) and abs(r["E"] - zero["E"]) < 1e-8
    got = step(ctx, 0.9 * rho)
    ctx.close()
    assert abs(got["E"] - ref["E"]) < 1e-8
