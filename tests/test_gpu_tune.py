"""What the section autotuner reports and what it remembers, where tiles of
sibling lines (a layout without a tile shape) compete with tiles of lines."""
import pytest
import torch

from paper_1404_0743_amd import pentago as P

pytestmark = pytest.mark.gpu


def counts_of(text):
    return tuple((int(text[2 * j]), int(text[2 * j + 1])) for j in range(4))


def empty_tables(counts):
    """Child tables in which every position is lost, and an output."""
    ch = [None] * 4
    for j in range(4):
        if sum(counts[j]) < 9:
            n = P.pentago_section_shape(P.pentago_child_section(counts, j))[1]
            ch[j] = torch.zeros((n, 8), dtype=torch.int64, device="cuda")
    return ch, torch.empty((P.pentago_section_shape(counts)[1], 8), dtype=torch.int64, device="cuda")


def best_ms(fn, reps=20):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    fn()
    times = []
    for _ in range(reps):
        a.record()
        fn()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def test_reported_time_is_that_of_the_reported_shape():
    """1,047,816 entries of 34 stones, two quadrants with empty cells: sibling
    tiles take two thirds of the time of the best tiles of lines."""
    counts = counts_of("63531853")
    ch, out = empty_tables(counts)
    print("autotune", counts, flush=True)
    shape, reported = P.pentago_autotune_section(counts, ch, out)
    assert P.pentago_debug_layout(counts)[1]
    lines = best_ms(lambda: P.pentago_solve_section_shape(counts, ch, out, **shape))
    siblings = best_ms(lambda: P.pentago_solve_section(counts, ch, out))
    print(shape, reported, lines, siblings, flush=True)
    assert siblings < 0.8 * lines
    assert abs(reported - lines) < 0.5 * (lines - siblings)


def test_equal_extents_with_other_runs_keep_their_layout():
    """Two sections of equal extents, staged quadrant and child lines, whose
    sibling quadrants are classes of exchanged colours with other runs: tuning
    the one, which has too many sibling tiles, says nothing of the other."""
    one, other = counts_of("08436372"), counts_of("80433627")
    assert P.pentago_section_shape(one)[0] == P.pentago_section_shape(other)[0]
    assert not P.pentago_debug_layout(one)[1] and P.pentago_debug_layout(other)[1]
    ch, out = empty_tables(one)
    print("autotune", one, flush=True)
    P.pentago_autotune_section(one, ch, out)
    assert P.pentago_debug_layout(other)[1]
