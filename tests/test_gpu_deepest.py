"""Roots with 9 and 10 empty cells in batches too large for a workgroup per
board: their own launch, whose workgroups without a layer slot, or with no such
root left, take roots with 8 empty cells.  Every result against the minimax
oracle, from outputs filled beforehand with a value no table holds."""
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
    pentago.pentago_init()
    return pentago


@pytest.fixture(scope="module")
def roots():
    """Boards with 10, 9, 8 and 5 empty cells and their tables."""
    boards = {e: I.random_play_boards(n, 36 - e, 36 - e, seed=900 + e) for e, n in ((10, 2), (9, 2), (8, 3), (5, 3))}
    return {e: (b, O.minimax_tables(b)) for e, b in boards.items()}


def batch(roots, counts, seed):
    """counts[e] boards of each size in random order, and their tables."""
    parts = [(roots[e][0][np.arange(n) % len(roots[e][0])], roots[e][1][np.arange(n) % len(roots[e][0])])
             for e, n in counts.items() if n]
    boards, want = (np.concatenate(x) for x in zip(*parts))
    order = np.random.default_rng(seed).permutation(len(boards))
    return boards[order], want[order]


def codes(P, boards):
    return torch.from_numpy(P.boards_to_codes(boards).view(np.int16).copy()).cuda()


# fewer roots of 9 and 10 empty cells than layer slots (64 without allocation,
# 512 else), as many, one more, several rounds; with and without roots of 8
COUNTS = [(1, 0), (1, 300), (63, 300), (64, 1), (65, 700), (511, 3), (512, 0), (513, 900), (1100, 257), (0, 600)]


@pytest.mark.parametrize("deep,eights", COUNTS)
def test_binned_deepest_roots(P, roots, deep, eights):
    boards, want = batch(roots, {10: deep // 2, 9: deep - deep // 2, 8: eights, 5: 280}, 7 * deep + eights)
    dev = codes(P, boards)
    for call, fill in ((P.pentago_eval_batch, -1), (P.pentago_eval_batch_noalloc, -2)):
        print(call.__name__, "9-10 empty cells", deep, "8", eights, flush=True)
        out = torch.full((len(boards), 8), fill, dtype=torch.int64, device="cuda")
        call(dev, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint64), want)


def best_ms(fn, reps=7):
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


def test_roots_of_eight_do_not_wait_for_the_deepest(P, roots):
    """The allocation-free call has layer slots for 64 workgroups: the others
    solve the roots with 8 empty cells meanwhile.  Together they take less than
    one launch after the other would (2000 deepest roots fill 2.4 ms on 64
    workgroups, 20,000 of the others 0.7 ms by themselves)."""
    ms = {}
    for name, counts in (("deepest", {10: 1000, 9: 1000}), ("eights", {8: 20000}),
                         ("both", {10: 1000, 9: 1000, 8: 20000})):
        boards, _ = batch(roots, counts, 5)
        dev = codes(P, boards)
        out = torch.empty((len(boards), 8), dtype=torch.int64, device="cuda")
        ms[name] = best_ms(lambda: P.pentago_eval_batch_noalloc(dev, out))
    print(ms, flush=True)
    assert ms["both"] < ms["deepest"] + 0.5 * ms["eights"], ms


@pytest.fixture
def threads(P):
    """Sets the threads per root; those from before come back at the end."""
    kept = P.pentago_debug_eval_threads()
    yield P.pentago_debug_eval_threads
    P.pentago_debug_eval_threads(kept)


@pytest.mark.parametrize("deep", (256, 512))
@pytest.mark.parametrize("eight", (256, 512))
def test_every_workgroup_size(P, roots, threads, deep, eight):
    threads((deep, eight, 768 - eight))
    boards, want = batch(roots, {10: 33, 9: 70, 8: 401, 5: 9}, deep + eight)
    dev = codes(P, boards)
    for call, fill in ((P.pentago_eval_batch, -1), (P.pentago_eval_batch_noalloc, -2)):
        print(call.__name__, "threads", deep, eight, flush=True)
        out = torch.full((len(boards), 8), fill, dtype=torch.int64, device="cuda")
        call(dev, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint64), want)


def test_autotuner_needs_roots_to_time(P, roots, threads):
    """A few boards take a launch without these sizes, and roots of 5 empty
    cells have none: tuning on them chooses nothing."""
    for counts in ({8: 3, 5: 7}, {5: 3000}):
        boards, _ = batch(roots, counts, 1)
        dev = codes(P, boards)
        out = torch.empty((len(boards), 8), dtype=torch.int64, device="cuda")
        for size in ((256, 256, 512), (512, 256, 256), (256, 512, 512), (512, 512, 256)):
            print("autotune", counts, size, flush=True)
            threads(size)
            got, ms = P.pentago_autotune_eval(dev, out)
            assert ms > 0 and got == size[1:]
            assert P.pentago_debug_eval_threads() == size
