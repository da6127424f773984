"""Deep solves of several sizes from several threads, each on its own stream:
their launches take different amounts of LDS of the same kernels."""
import threading

import numpy as np
import pytest
import torch

from paper_1404_0743_amd import inputs as I
from paper_1404_0743_amd import pentago as P

pytestmark = pytest.mark.gpu


def test_deep_solves_from_several_threads():
    boards = {e: P.boards_to_codes(I.random_play_boards(1, 36 - e, 36 - e, seed=70 + e))[0] for e in (13, 15, 16, 17)}
    want = {}
    for e, code in boards.items():
        out = torch.zeros(8, dtype=torch.int64, device="cuda")
        P.pentago_eval_deep(code, out)
        torch.cuda.synchronize()
        want[e] = out.cpu().numpy()
    wrong = []

    def solve(e):
        stream = torch.cuda.Stream()
        out = torch.empty(8, dtype=torch.int64, device="cuda")
        for k in range(10):
            with torch.cuda.stream(stream):
                out.fill_(-1)
            P.pentago_eval_deep(boards[e], out, stream)
            stream.synchronize()
            if not np.array_equal(out.cpu().numpy(), want[e]):
                wrong.append((e, k))

    print("deep solves from 4 threads", flush=True)
    threads = [threading.Thread(target=solve, args=(e,)) for e in boards]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
