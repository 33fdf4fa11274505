"""The whole-line FP64 solves that share the one-pass solve's launch: block
sizes down to one thread, lines shorter than a chunk of the sweeps, plans whose
every block takes the dropped system, and the mixed set of low wavenumbers."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


# (ny, n_parts, lines_per_block): 1 thread per block; 2 rows (the mean line keeps
# one); 2 partitions (all blocks dropped) and 8 + 1 rows; sweeps of 8k and 8k + 1
# rows; a padded last partition; the largest line
@pytest.mark.parametrize("ny,parts,lb", [(4, 1, 1), (2, 1, 3), (2, 2, 1), (9, 3, 1), (24, 2, 8), (64, 4, 0),
                                         (65, 0, 0), (130, 0, 0), (1024, 0, 0)])
def test_mean_line_matches_the_oracle(ny, parts, lb):
    from paper_2104_08863_amd.api import Plan
    nx, nz = 8, 6
    yf = synth.tanh_faces(ny, 1.5)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, n_parts=parts, lines_per_block=lb)
    rng = np.random.default_rng(ny)
    fh = rng.standard_normal((nx // 2 + 1, ny, nz)) + 1j * rng.standard_normal((nx // 2 + 1, ny, nz))
    box = O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)
    ref = O.solve_mean_line(torch.tensor(fh[0, :, 0]), box).numpy()
    got = pl.solve_spectral(torch.tensor(fh, device="cuda"))
    inplace = torch.tensor(fh, device="cuda")
    pl.solve_spectral(inplace, out=inplace)
    assert torch.equal(got, inplace)
    # two backward-stable solvers of the same line: a few eps times its
    # condition number, the ratio of the largest to the smallest nonzero eigenvalue
    a, c = (t.numpy() for t in O.y_coefficients(box))
    ev = np.sort(np.abs(np.linalg.eigvals(np.diag(a + c) - np.diag(a[1:], -1) - np.diag(c[:-1], 1))))
    bound = 8 * EPS * ev[-1] / ev[1] + 1e-13
    line = got[0, :, 0].cpu().numpy()
    assert np.linalg.norm(line - ref) <= bound * np.linalg.norm(ref)


def test_mixed_low_wavenumbers_are_fp64_lines():
    """Every special line of a mixed plan equals the FP64 line solve of its
    FP32 right-hand side, rounded once (and the kx = kz = 0 line its gauge)."""
    from paper_2104_08863_amd.api import Plan
    nx, ny, nz = 32, 48, 24
    yf = synth.tanh_faces(ny, 2.0)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, precision="mixed")
    rng = np.random.default_rng(5)
    fh = (rng.standard_normal((nx // 2 + 1, ny, nz)) + 1j * rng.standard_normal((nx // 2 + 1, ny, nz))).astype(np.complex64)
    got = pl.solve_spectral(torch.tensor(fh, device="cuda")).cpu().numpy()
    box = O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)
    ref = O.solve_spectral(torch.tensor(fh.astype(np.complex128)).permute(1, 2, 0), box).permute(2, 0, 1).numpy()
    for kx in range(4):
        for kz in range(nz):
            if min(kz, nz - kz) < 4:
                e = np.abs(got[kx, :, kz] - ref[kx, :, kz]).max() / np.abs(ref[kx, :, kz]).max()
                assert e <= np.finfo(np.float32).eps, (kx, kz, e)   # half an ulp per part, and FP64 round-off


# rows either side of the lanes' 1, 3 and 5 rows (the mean line has one row less)
@pytest.mark.parametrize("ny", [3, 63, 66, 128, 129, 192, 193, 194, 320, 322])
def test_special_lines_at_the_edges_of_the_lanes_rows(ny):
    """Any block size gives the same bits: a launch of their own beside blocks
    of less than one wave, and blocks of more than one wave.  The values are the
    oracle's within the bound of the first test, with a factor log2(64) for the
    depth of the scan."""
    from paper_2104_08863_amd.api import Plan
    nx, nz = 8, 6
    yf = synth.tanh_faces(ny, 1.5)
    parts = next(p for p in range(1, 65) if -(-ny // p) in (1, 2, 3, 4, 6, 8, 12, 16) and (p - 1) * -(-ny // p) < ny)
    rng = np.random.default_rng(ny)
    fh = rng.standard_normal((nx // 2 + 1, ny, nz)) + 1j * rng.standard_normal((nx // 2 + 1, ny, nz))
    box = O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)
    ref = O.solve_mean_line(torch.tensor(fh[0, :, 0]), box).numpy()
    a, c = (t.numpy() for t in O.y_coefficients(box))
    ev = np.sort(np.abs(np.linalg.eigvals(np.diag(a + c) - np.diag(a[1:], -1) - np.diag(c[:-1], 1))))
    lines = []
    for lb in (1, -(-128 // parts)):
        pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, n_parts=parts, lines_per_block=lb)
        lines.append(pl.solve_spectral(torch.tensor(fh, device="cuda"))[0, :, 0].cpu().numpy())
    assert np.array_equal(lines[0], lines[1])
    assert np.linalg.norm(lines[0] - ref) <= (6 * 8 * EPS * ev[-1] / ev[1] + 1e-13) * np.linalg.norm(ref)
