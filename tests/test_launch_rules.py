"""Host-side launch rules (cf_rules.h), on the CPU."""
import pytest

from paper_2104_08863_amd import _lib as L


@pytest.fixture(scope="module")
def H():
    return L.hostlib()


def single_step_graphs(nsteps, every):
    """Distinct graphs of a loop that replays one step at a time, by parity and
    with or without statistics."""
    return len({(k % 2, every > 0 and (k + 1) % every == 0) for k in range(nsteps)})


def test_alternating_loops_keep_their_graphs(H):
    """Loops in turn that fitted a cache of eight single-step graphs fit the plan's
    cache of one- and two-step graphs."""
    for nsteps in range(1, 64):
        for every in range(0, 16):
            mine, single = H.cfh_loop_graphs(nsteps, every), single_step_graphs(nsteps, every)
            assert mine <= 5
            assert (8 // single) * mine <= H.cfh_max_graphs(), (nsteps, every)
