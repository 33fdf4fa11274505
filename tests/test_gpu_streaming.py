"""The wall-normal solve of spectra large enough to be streamed (non-temporal
loads and stores) against the y-slab passes, which never are."""
import math

import pytest
import torch

from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu


# 2052 MiB of FP64 and 1026 MiB of FP32 spectrum, just past the sizes from which
# the one-pass solve streams; the FP64 plan drops most lines, drop_tol = 0 none
@pytest.mark.parametrize("nx,ny,nz,precision,drop_tol", [(1024, 512, 512, "fp64", -1.0), (1024, 512, 512, "fp64", 0.0),
                                                         (1024, 256, 1024, "mixed", -1.0)])
def test_streamed_solve_equals_the_slab_passes(nx, ny, nz, precision, drop_tol):
    from paper_2104_08863_amd.api import Plan
    pl = Plan(nx, ny, nz, 4 * math.pi, 2 * math.pi, synth.tanh_faces(ny, 2.5), precision=precision, drop_tol=drop_tol)
    assert (pl.info()["n_dropped_lines"] > 0) == (precision == "fp64" and drop_tol < 0)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(ny)
    fh = torch.randn(pl.spec_shape, dtype=pl.spec_dtype, device="cuda", generator=gen)
    ref = pl.solve_spectral_slabs(fh, 2)
    assert torch.equal(pl.solve_spectral(fh), ref)
    pl.solve_spectral(fh, out=fh)
    assert torch.equal(fh, ref)
