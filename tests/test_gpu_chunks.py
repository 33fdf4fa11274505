"""The marching stencils over the chunk lengths their launches choose: one-plane
chunks, a shorter last chunk, the longest chunks, tiles cut by the box in x and
z, and walls in the first and the last chunk."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu

# 2 and 3 planes (every plane at a wall); one-plane chunks; chunks of several
# planes with a remainder; x and z cut in mid tile; enough columns for the
# longest chunks of the split stages and the transposed stencil
GRIDS = [(4, 2, 2, 1.0), (8, 3, 4, 1.0), (64, 37, 16, 2.0), (96, 70, 48, 2.5), (256, 45, 96, 2.0), (512, 67, 384, 2.0)]


def rel(a, b):
    return float((a - b).norm() / b.norm())


def fields(nx, ny, nz, yf, dtype):
    q = [torch.tensor(t).to(dtype) for t in synth.perturbed_poiseuille(nx, ny, nz, yf, seed=nx + ny)]
    lam = [torch.tensor(t).to(dtype) for t in synth.random_directions(nx, ny, nz, seed=ny)]
    return q, lam


# the stencils' values are sums of about 100 products: eps times a few units
# relative to the result's norm (1e-13, 1e-6 in FP32); the transposed stencil
# cancels between neighbours that differ by O(1) times 1/dx^2 (one digit more)
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("mixed", 1e-6)])
@pytest.mark.parametrize("nx,ny,nz,gamma", GRIDS)
def test_stencils_match_the_oracle(nx, ny, nz, gamma, precision, tol):
    from paper_2104_08863_amd.api import Plan
    yf = synth.tanh_faces(ny, gamma)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, precision=precision, step=True)
    box = O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)
    q, lam = fields(nx, ny, nz, yf, pl.state_dtype)
    dt, nu = 1e-4, 1 / 550
    ref = O.rk2_predictor(*(t.double() for t in q), box, dt, nu, 3 * nu)
    g = [t.cuda() for t in q]
    fused = pl.rk2_predictor(*g, dt, nu, 3 * nu)
    lg = [t.cuda() for t in lam]
    adj = pl.rhs_adjoint(*g, *lg, nu)
    split = pl.rk2_predictor(*g, dt, nu, 3 * nu, out=tuple(g))
    for a, b, want in zip(fused, split, ref):
        if float(want.norm()) > 0:
            assert rel(a.cpu().double(), want) <= tol and rel(b.cpu().double(), want) <= tol
    assert bool((fused[1][-1] == 0).all()) and bool((split[1][-1] == 0).all())
    if nx * ny * nz > 2_000_000:
        return  # the oracle's gradient of the largest grid adds nothing the smaller ones lack
    qt = [t.double().requires_grad_(True) for t in q]
    want = torch.autograd.grad(O.momentum_rhs(*qt, box, nu, 0.3), qt, [t.double() for t in lam])
    for a, b in zip(adj, want):
        if float(b.norm()) > 0:
            assert rel(a.cpu().double(), b) <= 10 * tol
    assert bool((adj[1][-1] == 0).all())
