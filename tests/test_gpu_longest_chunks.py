"""The marching stencils in chunks of the most planes they take, with a shorter
last chunk.  A field that repeats in z many times fills such a grid; every copy
of the result must be the result on one period, whose chunks are short, and that
one the oracle's."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2104_08863_amd import _lib as L
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu

def chunk(nx, ny, nz, tx, tz, blocks_per_cu, most, extra):
    """Planes per chunk on 256 CUs with tiles of tx x tz columns."""
    return L.hostlib().cfh_chunk_planes(-(-nx // tx) * -(-nz // tz), ny, 256 * blocks_per_cu, most, extra)


def plans(nx, ny, nz, precision, copies):
    from paper_2104_08863_amd.api import Plan
    yf = synth.tanh_faces(ny, 2.0)
    small = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, precision=precision, step=True)
    large = Plan(nx, ny, nz * copies, 2 * np.pi, np.pi * copies, yf, precision=precision, step=True)
    q = [torch.tensor(t).to(small.state_dtype).cuda() for t in synth.perturbed_poiseuille(nx, ny, nz, yf, seed=ny)]
    lam = [torch.tensor(t).to(small.state_dtype).cuda() for t in synth.random_directions(nx, ny, nz, seed=ny)]
    return small, large, q, lam, O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)


def rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


def check_copies(large, small, tol):
    for a, b in zip(large, small):
        for part in a.split(b.shape[1], dim=1):
            assert rel(part, b) <= tol


def repeat(q, copies):
    return [t.repeat(1, copies, 1) for t in q]


# split stages (64 x 8 tiles, three blocks per CU) and transposed stencil (64 x 4,
# three blocks; FP32 128 x 4, two): 62 planes in chunks of 32 and 30.  Tolerances
# as for the stencils on other grids: a few units of eps in sums of about 100
# products, ten times that where neighbours cancel
@pytest.mark.parametrize("precision,copies,tol", [("fp64", 8, 1e-13), ("mixed", 16, 1e-6)])
def test_chunks_of_32_planes(precision, copies, tol):
    nx, ny, nz = 256, 62, 96
    adj = (64, 4, 3) if precision == "fp64" else (128, 4, 2)
    assert chunk(nx, ny, nz * copies, 64, 8, 3, 32, 2) == 32 and chunk(nx, ny, nz * copies, *adj, 32, 2) == 32
    assert chunk(nx, ny, nz, 64, 8, 3, 32, 2) < 32 and chunk(nx, ny, nz, *adj, 32, 2) < 32
    small, large, q, lam, box = plans(nx, ny, nz, precision, copies)
    dt, nu = 1e-4, 1 / 550
    big = repeat(q, copies)
    adj_large = large.rhs_adjoint(*big, *repeat(lam, copies), nu)
    adj_small = small.rhs_adjoint(*q, *lam, nu)
    qt = [t.cpu().double().requires_grad_(True) for t in q]
    want = torch.autograd.grad(O.momentum_rhs(*qt, box, nu, 0.3), qt, [t.cpu().double() for t in lam])
    for a, b in zip(adj_small, want):
        assert rel(a.cpu(), b) <= 10 * tol
    check_copies(adj_large, adj_small, 10 * tol)
    ref = O.rk2_predictor(*(t.cpu().double() for t in q), box, dt, nu, 3 * nu)
    split_large = large.rk2_predictor(*big, dt, nu, 3 * nu, out=tuple(big))
    split_small = small.rk2_predictor(*q, dt, nu, 3 * nu, out=tuple(q))
    for a, b in zip(split_small, ref):
        assert rel(a.cpu(), b) <= tol
    check_copies(split_large, split_small, tol)


# fused pass, FP64 (64 x 16 tiles, one block per CU): 250 planes in chunks of 128 and 122
def test_fused_chunks_of_128_planes():
    nx, ny, nz, copies = 256, 250, 128, 8
    assert chunk(nx, ny, nz * copies, 64, 16, 1, 128, 4) == 128 and chunk(nx, ny, nz, 64, 16, 1, 128, 4) < 128
    small, large, q, _, _ = plans(nx, ny, nz, "fp64", copies)
    dt, nu = 1e-4, 1 / 550
    fused_small = small.rk2_predictor(*q, dt, nu, 3 * nu)
    check_copies(large.rk2_predictor(*repeat(q, copies), dt, nu, 3 * nu), fused_small, 1e-13)
    # the split stages of the same field, in other chunks
    for a, b in zip(fused_small, small.rk2_predictor(*q, dt, nu, 3 * nu, out=tuple(q))):
        assert rel(a, b) <= 1e-13
