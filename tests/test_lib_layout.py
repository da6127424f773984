"""CPU checks of the layout a single section's sweep takes when nothing was
tuned, at sections whose layouts were timed against one another: the layout
that another rule would take there was slower by the factor noted."""
import pytest

from paper_1404_0743_amd import inputs as I
from paper_1404_0743_amd import pentago as P


def counts_of(text):
    return tuple((int(text[2 * j]), int(text[2 * j + 1])) for j in range(4))


# 512 threads took 1.9, 1.6, 1.4, 1.4, 1.3, 1.3 and 1.25 times as long
THROUGH_SYMMETRY = ["54459008", "07544481", "62635418", "53177036", "36623663", "50454536", "44078144"]


@pytest.mark.parametrize("counts", THROUGH_SYMMETRY)
def test_staged_representative_takes_256_threads(counts):
    shape, siblings = P.pentago_debug_layout(counts_of(counts), reps=True)
    assert not siblings
    assert shape["threads"] == 256 and shape["order"] == 0
    assert 1 <= shape["lines"] <= 8


def test_layouts_are_in_range():
    """Every layout stays inside what pentago_solve_section_shape accepts."""
    for stones in (32, 33, 34, 35):
        for s in I.all_sections(stones)[::17]:
            for reps in (False, True):
                shape, siblings = P.pentago_debug_layout(s, reps)
                assert shape["threads"] in (256, 512) and shape["order"] in (0, 1)
                assert 1 <= shape["lines"] <= (10 if siblings else 8)


@pytest.mark.parametrize("counts,lines,threads", [
    ("62364345", 2, 512),   # 318 patterns and 160 children to a line: one line took 1.3 times as long
    ("34454563", 2, 512),   # the same, 1.26
    ("34632763", 2, 512),   # the same, 1.12
    ("70452635", 8, 256),   # 80 parents to a tile: 512 threads took 1.08
    ("36443660", 8, 512),   # 176 parents to a tile: 256 threads took 1.16
    ("72450663", 8, 512),   # the same, 1.41
])
def test_plain_lines(counts, lines, threads):
    shape, siblings = P.pentago_debug_layout(counts_of(counts))
    assert not siblings
    assert shape == {"lines": lines, "threads": threads, "order": 1}


@pytest.mark.parametrize("counts,want", [
    ("63810835", True),     # 25,000 entries, a few hundred tiles: lines took 3 times as long
    ("63531853", True),     # 1,047,816 entries, 1452 tiles: 1.5
    ("71074553", False),    # 771,120 entries in 12,240 tiles: siblings took 1.3 times as long
    ("35703645", False),    # 942,480 entries in 14,960 tiles: 1.25
    ("70442745", False),    # 544,000 entries in 10,200 tiles: 1.3
    ("72545307", False),    # 428,400 entries in 5440 tiles: 1.1
    ("07634462", False),    # beyond 2^20 entries
])
def test_sibling_tiles_where_they_are_few(counts, want):
    assert P.pentago_debug_layout(counts_of(counts))[1] == want
