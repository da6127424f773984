"""The work a program has this library do, as cases that can be timed: sweeps
of single sections, of layers and of parts of a whole slice, endgame batches,
deep positions and the query server, each through its public entry point.

A case is a dict of plain values:
  kind "section"  one pentago_solve_section (d4: children held as their
                  representatives, pentago_solve_section_d4; tuned: its tile
                  shape picked by pentago_autotune_section beforehand)
  kind "layer"    `sections` sections of one slice (inputs.pick_layer_sections
                  with positions in [lo, hi]) as one batch: mode "graph" is a
                  SweepPlan replayed from its graph with a tuned tile shape,
                  mode "batch" one pentago_solve_sections call
  kind "slice"    every `step`-th D4-minimal section of a slice, from number
                  `first`, over the representatives of the slice above
                  (pentago_solve_sections_d4, as slices.solve_slice does)
  kind "endgame"  `boards` boards with lo..hi stones: pentago_eval_batch
  kind "deep"     one board with `stones` stones: pentago_eval_deep, or with
                  parity 0 or 1 pentago_eval_deep_parity
  kind "serve"    `queries` queries at once to a Server, half of them in its
                  resident sections and half random boards of lo..hi stones

Sections are written as eight digits, black and white stones per quadrant.
Child tables are seeded random valid tables (win inside not-lose, equal at
rotations that a symmetric quadrant pattern cannot tell apart): a solved
table of fixed counts would be the same for every seed.  Boards are seeded
random placements without a five.
"""
import functools
import math

import numpy as np
import torch

from paper_1404_0743_amd import inputs as I
from paper_1404_0743_amd import pentago as P

DEV = "cuda"


def listed():
    return [
        # one small section in the middle of a chain (the smallest sweep: launches count)
        {"name": "section34_small", "kind": "section", "counts": "63810835", "d4": False, "tuned": False},
        # one section with three empty cells in three quadrants, without tuning
        {"name": "section33", "kind": "section", "counts": "26355471", "d4": False, "tuned": False},
        # the 36 -> 35 sweep of bench.py: 6,288,640 entries, tuned as there
        {"name": "section35_headline", "kind": "section", "counts": "54455444", "d4": False, "tuned": True},
        # the 64-section layers of bench_extra.py: replayed plan, and one batched call
        {"name": "layer34_graph", "kind": "layer", "stones": 34, "sections": 64, "lo": 1e4, "hi": 2e8, "mode": "graph"},
        {"name": "layer33_batch", "kind": "layer", "stones": 33, "sections": 64, "lo": 1e4, "hi": 2e8, "mode": "batch"},
        # a sixth of the whole-slice sweep of slice 34 (the largest work here)
        {"name": "slice34_part", "kind": "slice", "stones": 34, "first": 0, "step": 6},
        # one position asked at a time
        {"name": "endgame_one", "kind": "endgame", "boards": 1, "lo": 29, "hi": 29},
        # the 4096 boards with 33 stones of bench_extra.py
        {"name": "endgame_4096", "kind": "endgame", "boards": 4096, "lo": 33, "hi": 33},
        # the 2^20 boards with 28..33 stones of bench_extra.py
        {"name": "endgame_2p20", "kind": "endgame", "boards": 1 << 20, "lo": 28, "hi": 33},
        # the deepest boards a batch takes: 9 and 10 empty cells
        {"name": "endgame_deepest", "kind": "endgame", "boards": 4096, "lo": 26, "hi": 27},
        # the 18-stone position of bench_extra.py
        {"name": "deep18", "kind": "deep", "stones": 18, "parity": -1},
        # a burst of queries to the server, lookups and searches one to one
        {"name": "serve_mixed", "kind": "serve", "queries": 32768, "lo": 26, "hi": 33},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(("section", "section", "section", "layer", "slice", "endgame", "endgame", "endgame", "deep",
                       "serve"))
    if kind == "section":
        stones = rng.choice((33, 34, 35))
        want = _log_uniform(rng, 2e3, 6.2e6)
        found = min(rng.sample(_sections(stones), 400), key=lambda s: abs(math.log(_entries(s) / want)))
        return {"kind": kind, "counts": "".join("%d%d" % q for q in found), "d4": rng.random() < 0.3,
                "tuned": rng.random() < 0.5}
    if kind == "layer":
        return {"kind": kind, "stones": rng.choice((33, 34, 35)), "sections": rng.randint(3, 64), "lo": 1e4,
                "hi": float(int(_log_uniform(rng, 1e6, 2e8))), "mode": rng.choice(("graph", "batch"))}
    if kind == "slice":
        step = rng.randint(8, 90)
        return {"kind": kind, "stones": 34, "first": rng.randrange(step), "step": step}
    if kind == "endgame":
        lo = rng.randint(26, 34)
        hi = min(35, lo + rng.randint(0, 5))
        most = 1 << (20 if lo >= 28 else 12)
        return {"kind": kind, "boards": int(_log_uniform(rng, 1, most)), "lo": lo, "hi": hi}
    if kind == "deep":
        return {"kind": kind, "stones": rng.randint(18, 24), "parity": rng.choice((-1, -1, 0, 1))}
    return {"kind": kind, "queries": int(_log_uniform(rng, 64, 32768)), "lo": rng.randint(26, 29), "hi": 33}


# ---------------------------------------------------------------- sections

@functools.lru_cache(None)
def _sections(stones):
    return I.all_sections(stones)


def _counts(text):
    return tuple((int(text[2 * j]), int(text[2 * j + 1])) for j in range(4))


@functools.lru_cache(None)
def _entries(counts):
    return P.pentago_section_shape(counts)[1]


def _children(counts):
    """The child section of each quadrant, None where the quadrant is full."""
    return [P.pentago_child_section(counts, j) if sum(counts[j]) < 9 else None for j in range(4)]


def _rep(counts):
    return P.pentago_section_standardize(counts)[0]


@functools.lru_cache(None)
def _layer(stones, sections, lo, hi):
    return tuple(I.pick_layer_sections(stones, sections, lo, hi))


@functools.lru_cache(None)
def _slice(stones, first, step):
    return tuple(P.pentago_slice_sections(stones)[first::step])


@functools.lru_cache(None)
def _symmetric(b, w):
    """{period: indices} of the patterns of a class that one turn or two turns
    leave unchanged."""
    other = ((b, w), (w, b), (0, 0), (0, 0))  # a section of valid counts that holds the class
    out = {1: [], 2: []}
    for i in range(P.pentago_section_shape(other)[0][0]):
        code = P.pentago_section_board(other, (i, 0, 0, 0))[0]
        q = np.array([code // 3 ** k % 3 for k in range(9)]).reshape(3, 3)
        if (np.rot90(q) == q).all():
            out[1].append(i)
        elif (np.rot90(q, 2) == q).all():
            out[2].append(i)
    return out


def _turned(w, j, k):
    """The set w (.., 4 words) with bit g at g + k along dimension j."""
    if j == 3:
        return torch.roll(w, k, -1)
    width, shift = (4, 16, 64)[j], (1, 4, 16)[j] * k
    ones = (1 << 64) - 1
    unit = sum(1 << s for s in range(0, 64, width))
    low = unit * ((1 << (width - shift)) - 1)      # bits that stay below the field's end
    signed = lambda m: m - (1 << 64) if m >> 63 else m  # noqa: E731
    up = (w & signed(low)) << shift
    down = ((w & signed(ones & ~low)) >> (width - shift)) & signed(unit * ((1 << shift) - 1))
    return up | down


def _offsets(shape, idx):
    """Blocked offsets of index vectors idx (four broadcastable tensors)."""
    B = [i >> 3 for i in idx]
    r = [i & 7 for i in idx]
    s = [(m - 8 * b).clamp(max=8) for m, b in zip(shape, B)]
    m1, m2, m3 = shape[1:]
    off = 8 * B[0] * (m1 * m2 * m3) + s[0] * 8 * B[1] * (m2 * m3) + s[0] * s[1] * 8 * B[2] * m3
    off = off + s[0] * s[1] * s[2] * 8 * B[3]
    return off + ((r[0] * s[1] + r[1]) * s[2] + r[2]) * s[3] + r[3]


def _sparse_words(n, k, gen):
    """(n, 4) random words with one bit in 2^k set."""
    draw = lambda: torch.randint(-(1 << 63), (1 << 63) - 1, (n, 4), generator=gen, device=DEV)  # noqa: E731
    words = draw()
    for _ in range(k - 1):
        words &= draw()
    return words


def _random_table(counts, gen):
    """A seeded random valid table of a section (entries x 8 int64)."""
    shape, n, _ = P.pentago_section_shape(counts)
    table = torch.empty((n, 8), dtype=torch.int64, device=DEV)
    # few losses (1 in 32) and ties (1 in 16): every value of a parent takes the
    # best of eight turns of every child, so more would make all parents equal
    loss, tie = _sparse_words(n, 5, gen), _sparse_words(n, 4, gen)
    table[:, 4:] = ~loss
    table[:, :4] = ~(loss | tie)
    del loss, tie
    grid = [torch.arange(m, device=DEV).reshape([-1 if k == j else 1 for k in range(4)]) for j, m in enumerate(shape)]
    for j in range(4):
        for period, which in _symmetric(*counts[j]).items():
            if not which:
                continue
            at = list(grid)
            at[j] = torch.tensor(which, device=DEV).reshape([-1 if k == j else 1 for k in range(4)])
            off = _offsets(shape, at).reshape(-1)
            rows = table[off].reshape(-1, 2, 4)
            kept = rows
            for k in range(period, 4, period):
                kept = kept & _turned(rows, j, k)
            table[off] = kept.reshape(-1, 8)
    return table


# ---------------------------------------------------------------- boards

def _has_five(b):
    """(n, 6, 6) bool -> (n,) bool: five in a row anywhere."""
    found = torch.zeros(len(b), dtype=torch.bool, device=b.device)
    for s in (0, 1):
        found |= b[:, :, s:s + 5].all(2).any(1) | b[:, s:s + 5, :].all(1).any(1)
        for t in (0, 1):
            sub = b[:, s:s + 5, t:t + 5]
            found |= sub.diagonal(dim1=1, dim2=2).all(1) | sub.flip(2).diagonal(dim1=1, dim2=2).all(1)
    return found


def _codes(boards):
    """(n, 6, 6) cells 0..2 -> (n, 4) int16 quadrant codes."""
    q = boards.reshape(-1, 2, 3, 2, 3).permute(0, 1, 3, 2, 4).reshape(-1, 4, 9).to(torch.int32)
    weight = 3 ** torch.arange(9, dtype=torch.int32, device=boards.device)
    return (q * weight).sum(2).to(torch.int16)


def _random_boards(n, lo, hi, gen):
    """n quadrant codes of boards with lo..hi stones and no five, in random order."""
    parts = []
    for stones in range(lo, hi + 1):
        left = n * (stones - lo + 1) // (hi - lo + 1) - n * (stones - lo) // (hi - lo + 1)
        black = (stones + 1) // 2
        value = torch.zeros(36, dtype=torch.uint8, device=DEV)
        value[:black] = 1
        value[black:stones] = 2
        while left > 0:
            perm = torch.rand((4 * left + 64, 36), generator=gen, device=DEV).argsort(1)
            b = value[perm].reshape(-1, 6, 6)
            b = b[~(_has_five(b == 1) | _has_five(b == 2))][:left]
            parts.append(_codes(b))
            left -= len(b)
    codes = torch.cat(parts)
    return codes[torch.randperm(len(codes), generator=gen, device=DEV)].contiguous()


def _resident_queries(sections, n, gen):
    """n quadrant codes of boards of the sections, every quadrant turned at random."""
    per = -(-n // len(sections))
    parts = []
    for s in sections:
        value = torch.zeros((4, 9), dtype=torch.uint8, device=DEV)
        for j, (b, w) in enumerate(s):
            value[j, :b] = 1
            value[j, b:b + w] = 2
        perm = torch.rand((per, 4, 9), generator=gen, device=DEV).argsort(2)
        cells = value.expand(per, 4, 9).gather(2, perm)
        parts.append((cells.to(torch.int32) * 3 ** torch.arange(9, dtype=torch.int32, device=DEV)).sum(2))
    codes = torch.cat(parts).to(torch.int16)
    return codes[torch.randperm(len(codes), generator=gen, device=DEV)[:n]]


# the sections resident in the server: one with 35 stones, two with 34
RESIDENT = ("54455444", "53274562", "63810835")


# ---------------------------------------------------------------- cases

def _job_sections(case):
    if case["kind"] == "layer":
        return _layer(case["stones"], case["sections"], case["lo"], case["hi"])
    return _slice(case["stones"], case["first"], case["step"])


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    state = {"case": case}
    if kind == "section":
        counts = _counts(case["counts"])
        below = _children(counts)
        tables = {}
        for c in below:
            if c is not None:
                key = _rep(c) if case["d4"] else c
                if key not in tables:
                    tables[key] = _random_table(key, gen)
        state["children"] = [None if c is None else tables[_rep(c) if case["d4"] else c] for c in below]
        state["counts"] = counts
        state["out"] = torch.empty((_entries(counts), 8), dtype=torch.int64, device=DEV)
        if case["tuned"] and not case["d4"]:
            P.pentago_autotune_section(counts, state["children"], state["out"])
    elif kind in ("layer", "slice"):
        sections = _job_sections(case)
        as_rep = kind == "slice"
        tables, jobs, at = {}, [], 0
        arena = torch.empty((sum(_entries(s) for s in sections), 8), dtype=torch.int64, device=DEV)
        for s in sections:
            ch = []
            for c in _children(s):
                key = None if c is None else _rep(c) if as_rep else c
                if key is not None and key not in tables:
                    tables[key] = _random_table(key, gen)
                ch.append(None if key is None else tables[key])
            jobs.append((s, ch, arena[at:at + _entries(s)]))
            at += _entries(s)
        state.update(jobs=jobs, out=arena)
        if case.get("mode") == "graph":
            P.pentago_autotune_sections(jobs)
            state["plan"] = P.SweepPlan(jobs)
    elif kind == "endgame":
        state["boards"] = _random_boards(case["boards"], case["lo"], case["hi"], gen)
        state["out"] = torch.empty((case["boards"], 8), dtype=torch.int64, device=DEV)
        state["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    elif kind == "deep":
        state["codes"] = _random_boards(1, case["stones"], case["stones"], gen)[0].tolist()
        state["out"] = torch.empty(8, dtype=torch.int64, device=DEV)
    else:
        n = case["queries"]
        sections = [_counts(t) for t in RESIDENT]
        asked = torch.empty((n, 4), dtype=torch.int16, device=DEV)
        asked[0::2] = _resident_queries(sections, n - n // 2, gen)
        asked[1::2] = _random_boards(n // 2, case["lo"], case["hi"], gen)
        state["codes"] = asked.cpu().numpy().view(np.uint16)
        state["arrivals"] = np.zeros(n)
        state["server"] = P.Server(memory_budget=4 << 30, max_inflight=1 << 20, max_batch=4096, streams=4)
        for s in sections:
            state["server"].add_section(s, _random_table(s, gen))
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "section":
        if case["d4"]:
            P.pentago_solve_section_d4(state["counts"], state["children"], state["out"])
        else:
            P.pentago_solve_section(state["counts"], state["children"], state["out"])
    elif kind == "layer":
        if case["mode"] == "graph":
            state["plan"].launch(graph=True)
        else:
            P.pentago_solve_sections(state["jobs"])
    elif kind == "slice":
        P.pentago_solve_sections_d4(state["jobs"])
    elif kind == "endgame":
        P.pentago_eval_batch(state["boards"], state["out"], state["status"])
        return state["out"], state["status"]
    elif kind == "deep":
        if case["parity"] < 0:
            P.pentago_eval_deep(state["codes"], state["out"])
        else:
            P.pentago_eval_deep_parity(state["codes"], case["parity"], state["out"])
    else:
        return state["server"].replay(state["codes"], state["arrivals"]).view(np.int64)
    return state["out"]


def _dag_ops(e):
    """32-bit operations on set words of one endgame root with e empty cells:
    per position 16 words (win and not-lose), each ORed over the children,
    rotated to its eight neighbours and combined with two five-sets."""
    return sum(math.comb(e, t) * math.comb(t, t // 2) * 16 * (e - t + 8 + 4) for t in range(e + 1))


def work(case):
    kind = case["kind"]
    if kind in ("section", "layer", "slice"):
        sections = [_counts(case["counts"])] if kind == "section" else _job_sections(case)
        as_rep = kind == "slice" or case.get("d4", False)
        below = {_rep(c) if as_rep else c for s in sections for c in _children(s) if c is not None}
        # a parent word takes at least its children, and each child word its eight neighbours
        ops = sum(16 * _entries(s) * (4 + sum(9 - sum(q) for q in s)) for s in sections)
        ops += sum(16 * 8 * _entries(c) for c in below)
        return {"bytes": 64 * (sum(map(_entries, sections)) + sum(map(_entries, below))), "flops": ops}
    if kind == "deep":
        return {"bytes": 8 + 64, "flops": _dag_ops(36 - case["stones"]) * (1 if case["parity"] < 0 else 0.5)}
    n = case["boards"] if kind == "endgame" else case["queries"]
    mean = sum(_dag_ops(36 - k) for k in range(case["lo"], case["hi"] + 1)) / (case["hi"] - case["lo"] + 1)
    if kind == "endgame":
        return {"bytes": n * (8 + 64), "flops": n * mean}
    # half of the queries read one 64-byte entry
    return {"bytes": n * (8 + 64) + n // 2 * 64, "flops": n // 2 * mean}


def exact(case, seed):
    """The outputs are sets of bits, compared bit for bit: there is no rounding
    that a wider computation could show."""
    return None
