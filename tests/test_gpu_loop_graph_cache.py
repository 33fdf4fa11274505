"""More recorded graphs than a plan keeps: the least recently used are dropped and
recorded again, and every replay equals the eager loop."""
import numpy as np
import pytest
import torch

from paper_2104_08863_amd import _lib as L
from paper_2104_08863_amd import synth

pytestmark = pytest.mark.gpu


def test_dropped_graphs_are_recorded_again():
    from paper_2104_08863_amd.api import Plan
    nx, ny, nz, nsteps, every = 32, 16, 24, 7, 3
    yf = synth.tanh_faces(ny, 2.0)
    pl = Plan(nx, ny, nz, 2 * np.pi, np.pi, yf, step=True)
    q = [torch.tensor(t).cuda() for t in synth.perturbed_poiseuille(nx, ny, nz, yf, seed=7)]
    per_set = L.hostlib().cfh_loop_graphs(nsteps, every)
    sets = L.hostlib().cfh_max_graphs() // per_set + 2      # together more than the plan keeps
    a = [[torch.empty_like(t) for t in q] for _ in range(2)]
    st = [torch.zeros(ny, 6, dtype=torch.float64, device="cuda") for _ in range(2)]
    for rep in range(2):
        for k in range(sets):
            out = []
            for m in range(2):      # from graphs, then eager
                for t, x in zip(a[0], q):
                    t.copy_(x)
                st[m].zero_()
                got = pl.run_steps(*a[0], nsteps, 1e-3 * (1 + 0.1 * k), 1 / 550, 3 / 550, work=tuple(a[1]),
                                   stats_every=every, stats=st[m], use_graph=m == 0)
                out.append([t.clone() for t in got])
            for x, y in zip(*out):
                assert torch.equal(x, y), (rep, k)
            assert torch.equal(st[0], st[1]), (rep, k)
