"""Slab counts and drop_parts given to a plan whose partition count is
automatic: counts that divide the even partitioning of ny (the fewest partitions
that divide it) are taken, whatever count is the cheapest on one device.  And a
plan tuned by measurement times what an untuned one would take, and the default
blocks of the FP32 partitions of 24 rows."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu


def make(ny, nx=32, nz=24, **kw):
    from paper_2104_08863_amd.api import Plan
    yf = synth.tanh_faces(ny, 2.0)
    return Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, **kw), O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)


def spectrum(pl, seed):
    rng = np.random.default_rng(seed)
    fh = rng.standard_normal(pl.spec_shape) + 1j * rng.standard_normal(pl.spec_shape)
    fh[0, :, 0].imag = 0.0
    return torch.tensor(fh, device="cuda")


# (ny, partitions of the even count): every divisor of it is a slab count.  45 =
# 15 x 3, 54 = 9 x 6, 56 = 7 x 8, 27 = 9 x 3; 97 rows pad: 49 x 2 pads one row
@pytest.mark.parametrize("ny,even", [(45, 15), (54, 9), (56, 7), (27, 9), (97, 49)])
def test_slab_counts_of_the_even_partitioning(ny, even):
    pl, box = make(ny)
    fh = spectrum(pl, ny)
    want = O.solve_spectral(fh.cpu().permute(1, 2, 0), box).permute(2, 0, 1).numpy()
    scale = np.abs(want).max(axis=1)
    counts = [g for g in range(1, even + 1) if even % g == 0 or pl.info()["n_parts"] % g == 0]
    for g in counts:
        got = pl.solve_spectral_slabs(fh, g)
        noalloc = torch.empty_like(fh)
        pl.solve_spectral_slabs_noalloc(fh, g, noalloc)
        assert torch.equal(got, noalloc), g
        if pl.info()["n_parts"] % g == 0:
            assert torch.equal(got, pl.solve_spectral(fh)), g
        # per line, the bound of the one-pass solve
        assert (np.abs(got.cpu().numpy() - want).max(axis=1) / scale).max() <= 1e-11, g


@pytest.mark.parametrize("ny,drop_parts", [(27, 3), (54, 9), (45, 5)])
def test_drop_parts_of_the_even_partitioning(ny, drop_parts):
    pl, box = make(ny, drop_parts=drop_parts)
    info = pl.info()
    assert info["drop_parts"] == drop_parts and info["n_parts"] % drop_parts == 0
    fh = spectrum(pl, ny)
    want = O.solve_spectral(fh.cpu().permute(1, 2, 0), box).permute(2, 0, 1).numpy()
    got = pl.solve_spectral(fh).cpu().numpy()
    assert (np.abs(got - want).max(axis=1) / np.abs(want).max(axis=1)).max() <= 1e-11


# 144 = 9 x 16 with blocks of 24 lines; 102 rows as 9 x 12, padded although 17 x 6
# divides; 65 * 96 lines make 260 blocks of 24
@pytest.mark.parametrize("ny", [144, 102])
def test_tuning_times_the_untuned_pair(ny):
    auto, _ = make(ny, 128, 96)
    pair = auto.info()["n_parts"], auto.info()["lines_per_block"]
    assert pair == (9, 24)
    pl, box = make(ny, 128, 96, tune_parts=True)
    rows = pl.partition_timings()
    assert len({r[:2] for r in rows}) == len(rows) and pair in {r[:2] for r in rows}
    best = min(rows, key=lambda r: r[2])
    assert (pl.info()["n_parts"], pl.info()["lines_per_block"]) == best[:2]
    f = torch.tensor(synth.uniform_rhs(128, ny, 96, seed=ny), device="cuda")
    p = pl.poisson_solve(f)
    same, _ = make(ny, 128, 96, n_parts=best[0], lines_per_block=best[1])
    assert torch.equal(p, same.poisson_solve(f))
    ref = O.poisson(f.cpu(), box)
    assert float((p.cpu() - ref).norm() / ref.norm()) <= 1e-12


# FP32 partitions of 24 rows: 32 lines per block from 13 to 16 of them, 16 either side
@pytest.mark.parametrize("parts,lb", [(11, 16), (13, 32), (14, 32), (15, 32), (16, 32), (32, 16)])
def test_block_of_the_24_row_partitions(parts, lb):
    ny = 24 * parts
    pl, _ = make(ny, precision="mixed")
    assert (pl.info()["n_parts"], pl.info()["rows_per_part"], pl.info()["lines_per_block"]) == (parts, 24, lb)
    other, _ = make(ny, precision="mixed", n_parts=parts, lines_per_block=8)
    fh = spectrum(pl, ny).to(torch.complex64)
    assert torch.equal(pl.solve_spectral(fh), other.solve_spectral(fh))
