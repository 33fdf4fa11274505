"""The dropped reduced system: which lines a plan says it drops and which its
solve drops, groups of several partitions, mixed precision, the y-slab finishing
pass, and plans whose every block drops (the special lines then go with the
dropped blocks' launch)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu


def make(nx, ny, nz, gamma, **kw):
    from paper_2104_08863_amd.api import Plan
    yf = synth.tanh_faces(ny, gamma)
    return Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, **kw), O.Box(nx, ny, nz, 2 * np.pi, np.pi, yf)


def spectrum(pl, seed):
    rng = np.random.default_rng(seed)
    fh = rng.standard_normal(pl.spec_shape) + 1j * rng.standard_normal(pl.spec_shape)
    fh[0, :, 0].imag = 0.0
    return torch.tensor(fh).to(pl.spec_dtype).cuda()


def dropped_lines(pl, box):
    """(nkx, nz): the lines whose block of lines_per_block consecutive lines lies
    wholly above the threshold; all False when the plan drops none."""
    info = pl.info()
    k2 = O.line_coefficients(box)[2].numpy().T.reshape(-1)
    ok = np.zeros(k2.size, dtype=bool)
    for b0 in range(0, k2.size, info["lines_per_block"]):
        s = slice(b0, b0 + info["lines_per_block"])
        ok[s] = info["n_dropped_lines"] > 0 and bool((k2[s] >= info["k2_threshold"]).all())
    assert ok.sum() == info["n_dropped_lines"]
    return ok.reshape(pl.nkx, pl.nz)


# at these tolerances the two systems agree to round-off but not to the bit, which
# shows the lines that took the dropped one
@pytest.mark.parametrize("precision,ny,tol", [("fp64", 64, 1e-15), ("mixed", 96, 1e-7)])
@pytest.mark.parametrize("given", ["default", "drop_tol", "drop_parts"])
def test_a_plan_drops_the_lines_it_reports(precision, ny, tol, given):
    kw = {"default": {}, "drop_tol": {"drop_tol": tol}, "drop_parts": {"drop_parts": 4}}[given]
    pl, box = make(128, ny, 128, 2.5, precision=precision, **kw)
    exact, _ = make(128, ny, 128, 2.5, precision=precision, drop_tol=0.0)
    assert exact.info()["n_dropped_lines"] == 0
    n = pl.info()["n_dropped_lines"]
    assert (n == 0) == (given == "default")
    fh = spectrum(pl, 1)
    differ = (pl.solve_spectral(fh) != exact.solve_spectral(fh)).any(dim=1).cpu().numpy()
    assert not (differ & ~dropped_lines(pl, box)).any()
    assert differ.sum() >= n / 2     # nearly every dropped line differs in some bit


def special_lines(pl):
    """(kx, kz) of the lines solved whole: kx = kz = 0, in mixed plans the 28 lowest."""
    if pl.precision == "fp64":
        return [(0, 0)]
    return [(kx, kz) for kx in range(4) for kz in range(pl.nz) if min(kz, pl.nz - kz) < 4]


def check_lines(pl, box, fh, groups):
    """Dropped lines against the oracle's dropped PDD of `groups` partitions, all
    others against Thomas; returns the largest difference of a dropped line from
    the exact solution in units of its bound."""
    eps = np.finfo(np.float64 if pl.precision == "fp64" else np.float32).eps
    got = pl.solve_spectral(fh).cpu().numpy().astype(np.complex128)
    f = fh.cpu().numpy().astype(np.complex128)
    a, c, k2 = O.line_coefficients(box)
    k2 = k2.numpy().T.copy()
    drop = dropped_lines(pl, box)
    assert 0 < drop.sum() < drop.size
    for kx, kz in special_lines(pl):
        drop[kx, kz] = False     # whole-line solves
    far = 0.0
    for want in (True, False):
        sel = np.argwhere(drop == want)
        sel = sel[(sel[:, 0] > 0) | (sel[:, 1] > 0)]
        kk = k2[sel[:, 0], sel[:, 1]]
        b = -(a + c)[:, None] - torch.tensor(kk)[None, :]
        d = torch.tensor(np.ascontiguousarray(f[sel[:, 0], :, sel[:, 1]].T))
        x = got[sel[:, 0], :, sel[:, 1]].T
        exact = O.thomas(a[:, None], b, c[:, None], d).numpy()
        ref = O.pdd_solve(a, b, c, d, groups, drop=True).numpy() if want else exact
        scale = np.abs(exact).max(0)
        # rounding a diagonal -(a + c) - k2 moves a line's dominance k2 by eps (a +
        # c), so two correct solvers differ by a few eps (1 + max(a + c) / k2)
        bound = 32 * eps * (1 + float((a + c).max()) / kk)
        assert (np.abs(x - ref).max(0) <= bound * scale).all(), want
        if want:
            far = (np.abs(x - exact).max(0) / scale / bound).max()
    return far


# groups of 4, 3, 2 and 1 partitions; tolerances loose enough for most blocks of the
# grid to drop and for the drop to show (FP32: to show above the bound)
@pytest.mark.parametrize("precision,ny,parts,groups,lb,tol", [
    ("fp64", 128, 16, 4, 8, 1e-4), ("fp64", 96, 12, 3, 8, 1e-4), ("fp64", 64, 8, 4, 8, 1e-4), ("fp64", 64, 4, 4, 16, 1e-4),
    ("mixed", 64, 16, 4, 8, 0.02), ("mixed", 96, 12, 4, 8, 0.02), ("mixed", 48, 8, 4, 8, 0.02), ("mixed", 96, 4, 4, 16, 0.02)])
def test_groups_match_the_dropped_pdd_of_the_oracle(precision, ny, parts, groups, lb, tol):
    pl, box = make(64, ny, 48, 1.0, precision=precision, n_parts=parts, drop_parts=groups, lines_per_block=lb,
                   drop_tol=tol)
    assert pl.info()["drop_parts"] == groups
    # the drop is visible: some line is further from the exact solution than round-off
    assert check_lines(pl, box, spectrum(pl, ny), groups) > 4


@pytest.mark.parametrize("precision,ny,parts,tol", [("fp64", 128, 8, 1e-4), ("fp64", 96, 12, 1e-4),
                                                    ("mixed", 192, 8, 0.005)])
def test_slabs_drop_as_the_one_pass_solve(precision, ny, parts, tol):
    pl, _ = make(64, ny, 48, 1.0, precision=precision, n_parts=parts, lines_per_block=8, drop_tol=tol)
    assert pl.info()["n_dropped_lines"] > 0
    fh = spectrum(pl, ny)
    ref = pl.solve_spectral(fh)
    for g in [d for d in range(1, parts + 1) if parts % d == 0]:
        assert torch.equal(pl.solve_spectral_slabs(fh, g), ref), g


# one and two partitions have no corner terms: every block drops, with 64 to 512
# threads; (2, 1) is a block of less than one wave, whose special lines go alone
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("parts,lb", [(1, 64), (2, 32), (2, 256), (2, 1)])
def test_special_lines_of_a_plan_whose_every_block_drops(precision, parts, lb):
    nx, nz, ny, gamma = 16, 12, 12 * parts, 1.5
    pl, box = make(nx, ny, nz, gamma, precision=precision, n_parts=parts, lines_per_block=lb, drop_tol=1e-15)
    exact, _ = make(nx, ny, nz, gamma, precision=precision, n_parts=parts, lines_per_block=lb)
    assert pl.info()["n_dropped_lines"] == pl.info()["n_lines"] and exact.info()["n_dropped_lines"] == 0
    fh = spectrum(pl, parts + lb)
    got = pl.solve_spectral(fh)
    other = exact.solve_spectral(fh)
    # the special lines do not depend on the launch that carries them
    for kx, kz in special_lines(pl):
        assert torch.equal(got[kx, :, kz], other[kx, :, kz]), (kx, kz)
    inplace = fh.clone()
    pl.solve_spectral(inplace, out=inplace)
    assert torch.equal(inplace, got)
    want = O.solve_spectral(fh.cpu().to(torch.complex128).permute(1, 2, 0), box).permute(2, 0, 1).numpy()
    err = np.abs(got.cpu().numpy() - want).max(axis=1) / np.abs(want).max(axis=1)
    a, c, k2 = O.line_coefficients(box)
    k2 = k2.numpy().T.copy()
    k2[0, 0] = (np.pi / 2) ** 2 / 2      # the mean line's smallest eigenvalue, halved
    eps = np.finfo(np.float64 if precision == "fp64" else np.float32).eps
    assert (err <= 32 * eps * (1 + float((a + c).max()) / k2)).all()
