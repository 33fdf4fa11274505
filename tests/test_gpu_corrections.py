"""The pressure-gradient corrections by pairs of points: rows of one pair or two
(the second value's neighbour is the row's own first), planes that end inside a
block, odd z lengths of a wave, and chunks of the fused statistics that end inside
a plane."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu


# FP64: a step and its adjoint on these grids are sums of at most some hundred
# products and a solve of condition below 1e4 (1e-10).  Mixed: the FP32 state and
# the FP32 terms of its stencils, 1e-5.
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("mixed", 1e-5)])
@pytest.mark.parametrize("nx,ny,nz", [(4, 8, 2), (6, 9, 3), (12, 16, 6), (48, 12, 24), (96, 8, 48)])
def test_step_statistics_and_adjoint_match_the_oracle(nx, ny, nz, precision, tol):
    from paper_2104_08863_amd.api import Plan
    yf = synth.tanh_faces(ny, 1.2)
    box = O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, precision=precision, adjoint=True)
    dt, nu = 1e-3, 1 / 550
    q = [torch.tensor(t).to(pl.state_dtype) for t in synth.perturbed_poiseuille(nx, ny, nz, yf, seed=nx)]
    lam = [torch.tensor(t).to(pl.state_dtype) for t in synth.random_directions(nx, ny, nz, seed=ny)]
    qt = [t.double().requires_grad_(True) for t in q]
    want = O.projection_step(*qt, box, dt, nu, 3 * nu)[:3]
    g = [t.cuda() for t in q]
    got = pl.projection_step(*g, dt, nu, 3 * nu)
    scale = float(want[0].detach().norm())
    for a, b in zip(got, want):
        assert float((a.double().cpu() - b.detach()).norm()) <= tol * scale
    st = torch.zeros(ny, 6, dtype=torch.float64, device="cuda")
    new = pl.run_steps(*[t.clone() for t in g], 1, dt, nu, 3 * nu, stats_every=1, stats=st)
    mean = torch.stack([t.double().mean(dim=(1, 2)) for t in new] + [t.double().square().mean(dim=(1, 2)) for t in new], 1)
    assert all(torch.equal(a, b) for a, b in zip(new, got))
    assert float((st - mean).abs().max()) <= 1e-13 * float(mean.abs().max())
    ref = torch.autograd.grad(want, qt, [t.double() for t in lam])
    adj = pl.projection_step_adjoint(*g, *[t.cuda() for t in lam], dt, nu, 3 * nu)
    scale = float(torch.cat([t.flatten() for t in ref]).norm())
    for a, b in zip(adj, ref):
        assert float((a.double().cpu() - b).norm()) <= tol * scale
