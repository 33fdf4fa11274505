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


@pytest.mark.parametrize("most,extra", [(32, 2), (128, 4)])
def test_chunk_lengths(H, most, extra):
    """Chunks are within their limits and within 4 % of the least rounds of blocks
    times planes; a grid of few columns fills the chip, one of many takes the
    longest chunks it can."""
    for ny in (1, 2, 3, 31, 32, 33, 62, 97, 128, 130, 250, 256, 1024):
        for cols in (1, 4, 64, 300, 768, 1536, 65536):
            for slots in (256, 512, 768):
                cost = lambda cy: -(-(cols * -(-ny // cy)) // slots) * (cy + extra)  # noqa: E731
                cy = H.cfh_chunk_planes(cols, ny, slots, most, extra)
                top = min(most, ny)
                assert 1 <= cy <= top
                least = min(cost(c) for c in range(1, top + 1))
                assert 100 * cost(cy) <= 104 * least
                assert all(100 * cost(c) > 104 * least for c in range(cy + 1, top + 1))
    assert H.cfh_chunk_planes(4, 64, 256, 128, 4) == 1       # four columns: one plane per block
    assert H.cfh_chunk_planes(65536, 64, 768, 32, 2) == 32


def test_rows_of_the_corrections_take_eight_blocks(H):
    """Rows of a multiple of 1024 points are whole blocks, a multiple of the 8 XCDs of
    them; a block is whole waves and at most 256 threads, a pair of points each."""
    for nx in [2 ** a for a in range(2, 13)] + [3 * 2 ** a for a in range(1, 11)]:
        th = H.cfh_correction_threads(nx)
        assert th % 64 == 0 and 64 <= th <= 256
        if nx % 1024 == 0:
            assert nx % (2 * th) == 0 and nx // (2 * th) % 8 == 0
