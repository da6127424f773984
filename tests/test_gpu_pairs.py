"""The pair solver of the endgame (two roots of as many empty cells solved side
by side) and the two ways a batch reaches it: without binning, a workgroup per
board, for batches of at most one board per CU, else through the bins of empty
cells.  Every result is compared bit for bit with the minimax oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1404_0743_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_1404_0743_amd import pentago
    torch.cuda.set_device(0)
    return pentago


def solve(P, boards):
    codes = torch.from_numpy(P.boards_to_codes(boards).view(np.int16).copy()).cuda()
    out = torch.full((len(boards), 8), -1, dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    P.pentago_eval_batch(codes, out, status)
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.uint64), int(status.item())


def distinct(e, n, seed):
    """n boards with e empty cells, some of them spread unevenly over the quadrants."""
    stones = 36 - e
    boards = I.random_placement_boards(n, (stones + 1) // 2, stones // 2, seed=seed)
    return boards


@pytest.mark.parametrize("e", range(9))
def test_pairs_and_odd_tails(P, e):
    """Batches above and below the size that goes without bins, even and odd,
    ending in a pair of one root and in a partly filled workgroup."""
    boards = distinct(e, 7 if e < 7 else 4, 700 + e)
    want = O.minimax_tables(boards)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for n in (1, 2, 5, cus, cus + 1, cus + 2, cus + 15, 2 * cus + 3):
        print("pairs, empty cells", e, "boards", n, flush=True)
        idx = np.arange(n) % len(boards)
        got, bad = solve(P, boards[idx])
        assert bad == 0
        assert np.array_equal(got, want[idx]), n


def test_one_quadrant_holds_the_empty_cells(P):
    """All eight empty cells in one quadrant, each quadrant in turn."""
    rng = np.random.default_rng(9)
    boards = []
    for q in range(4):
        cells = [6 * (3 * (q // 2) + k // 3) + 3 * (q % 2) + k % 3 for k in range(8)]
        rest = np.array([c for c in range(36) if c not in cells])
        rng.shuffle(rest)
        b = np.zeros(36, np.uint8)
        b[rest[:14]], b[rest[14:]] = 1, 2
        boards.append(b)
    boards = np.array(boards)
    want = O.minimax_tables(boards)
    idx = np.arange(600) % 4
    print("one quadrant", flush=True)
    got, bad = solve(P, boards[idx])
    assert bad == 0
    assert np.array_equal(got, want[idx])


@pytest.mark.parametrize("n", [8191, 8192, 8193])
def test_bins_at_the_size_where_one_workgroup_ends(P, n):
    """Mixed numbers of empty cells and invalid boards, binned by one
    workgroup or by many."""
    print("bins", n, flush=True)
    boards = np.concatenate([distinct(e, 3, 800 + e) for e in range(7)])
    want = O.minimax_tables(boards)
    bad_board = np.zeros((1, 36), np.uint8)
    boards = np.concatenate([boards, bad_board])
    want = np.concatenate([want, np.zeros((1, 8), np.uint64)])
    idx = np.random.default_rng(n).integers(0, len(boards), size=n)
    got, bad = solve(P, boards[idx])
    assert bad == int((idx == len(boards) - 1).sum())
    assert np.array_equal(got, want[idx])
