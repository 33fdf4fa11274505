"""Time loops replayed from graphs of one step, one step with statistics and two
steps, over step counts and statistics cadences that mix them in both parities."""
import numpy as np
import pytest
import torch

from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("every", [0, 1, 2, 3, 5])
def test_replays_equal_the_eager_loop(every, precision):
    from paper_2104_08863_amd.api import Plan
    nx, ny, nz = 16, 12, 8
    yf = synth.tanh_faces(ny, 1.5)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, precision=precision, step=True)
    q = [torch.tensor(t).to(pl.state_dtype).cuda() for t in synth.perturbed_poiseuille(nx, ny, nz, yf, seed=4)]
    sets = [[torch.empty_like(t) for t in q] for _ in range(4)]
    st = [torch.zeros(ny, 6, dtype=torch.float64, device="cuda") for _ in range(2)]
    p = [torch.empty(ny, nz, nx, dtype=torch.float64, device="cuda") for _ in range(2)]
    for nsteps in (1, 2, 3, 4, 5, 6, 7, 11, 7, 2):
        out = []
        for m in range(2):   # eager, then from graphs: each replay follows eager work
            for t, x in zip(sets[2 * m], q):
                t.copy_(x)
            st[m].zero_()
            out.append(pl.run_steps(*sets[2 * m], nsteps, 1e-3, 1 / 550, 3 / 550, work=tuple(sets[2 * m + 1]),
                                    stats_every=every, stats=st[m] if every else None, p=p[m], use_graph=m == 1))
        for a, b in zip(*out):
            assert torch.equal(a, b), nsteps
        assert torch.equal(st[0], st[1]) and torch.equal(p[0], p[1]), nsteps
