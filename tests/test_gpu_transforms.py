"""The FP64 transforms at every length whose radices or block shape depend on the
precision or the size of the spectrum: short and 3 * 2^a lengths in x and z, in
spectra below and above 160 MiB (one-wave and full blocks, cached and streamed),
and rows that do not fill a block."""
import numpy as np
import pytest
import torch

from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def check(nx, ny, nz, y_solver="pdd"):
    from paper_2104_08863_amd.api import Plan
    yf = synth.uniform_faces(ny)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, y_solver=y_solver)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx + 7 * nz)
    f = torch.randn(ny, nz, nx, dtype=torch.float64, device="cuda", generator=gen)
    ref = torch.fft.fft(torch.fft.rfft(f, dim=2), dim=1).permute(2, 0, 1).contiguous()
    got = pl.forward_spectral(f)
    # two stable FFTs of N points: each within a few eps log2(N) of the exact one
    bound = 4 * EPS * np.log2(nx * nz)
    assert float((got - ref).norm() / ref.norm()) <= bound
    back = pl.inverse_spectral(got)
    assert float((back - f).norm() / f.norm()) <= 2 * bound
    return pl, f


@pytest.mark.parametrize("nz", [2, 6, 12, 16, 24, 32, 48, 64, 96, 192, 384, 768, 1536])
@pytest.mark.parametrize("big", [False, True])
def test_z_lengths(nz, big):
    nx = 2048 if big else 256
    ny = max(2, -(-(10_600_000 if big else 20_000) // ((nx // 2 + 1) * nz)))
    if ny > 1024:
        pytest.skip("more rows than a line may have")
    check(nx, ny, nz)


# nz = 6 and 24: blocks of 8 and 16 rows that the plane does not fill
@pytest.mark.parametrize("nx", [4, 12, 32, 48, 64, 96, 128, 192, 384, 768, 1536, 3072])
@pytest.mark.parametrize("nz", [6, 24])
def test_x_lengths(nx, nz):
    check(nx, 5, nz)


@pytest.mark.parametrize("nx,ny,nz", [(64, 24, 12), (64, 96, 48), (256, 64, 384), (512, 192, 48), (64, 768, 96)])
def test_uniform_y_solve_equals_the_partitioned_one(nx, ny, nz):
    """The two solvers of a line differ by at most its
    condition number 1 / sin^2(pi / 2 ny) times eps."""
    pl, f = check(nx, ny, nz, y_solver="dct")
    from paper_2104_08863_amd.api import Plan
    other = Plan(nx, ny, nz, 2 * np.pi, np.pi, synth.uniform_faces(ny))
    a, b = pl.poisson_solve(f), other.poisson_solve(f)
    assert float((a - b).norm() / b.norm()) <= 2 * EPS / np.sin(np.pi / (2 * ny)) ** 2 + 1e-13
