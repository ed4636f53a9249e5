"""The waits between braid steps: every order that the data of a sequence of steps asks for follows from the waits that are made
(directly or through other streams' waits), for three streams and for triples that share one, and no wait is made that earlier
ones imply."""
import ctypes as C
import random

import numpy as np
import pytest

import paper_2510_27257_amd as stp

TRIPLES = {"abc": (0, 1, 2), "aab": (0, 0, 2), "aba": (0, 1, 0), "abb": (0, 1, 1), "aaa": (0, 0, 0)}


def plan(mbs, f_mb, b, w, through, slot_of):
    f = stp.lib().stp_braid_plan_joins
    f.restype = C.c_int
    waits = np.zeros(1 << 14, np.int64)
    keep = [np.ascontiguousarray(f_mb, np.int32), *(np.ascontiguousarray(a, np.uint8) for a in (b, w, through)), np.array(slot_of, np.int32)]
    n = f(len(f_mb), mbs, *(a.ctypes.data_as(C.c_void_p) for a in keep), waits.ctypes.data_as(C.c_void_p), len(waits))
    assert n >= 0
    return [(int(x) & 0xffff, int(x) >> 16 & 15, int(x) >> 20 & 15, int(x) >> 24) for x in waits[:n]]


@pytest.mark.parametrize("streams", list(TRIPLES))
@pytest.mark.parametrize("seed", range(20))
def test_waits_imply_every_needed_order_and_none_is_spare(seed, streams):
    rng = random.Random(seed)
    n, mbs, slot_of = 40, rng.choice([2, 3, 5]), TRIPLES[streams]
    density = rng.choice([0.2, 0.5, 0.9])
    f_mb = [rng.randrange(mbs) if rng.random() < density else -1 for _ in range(n)]
    # B and W work on other microbatches than the step's forward one (the two directions of one step share nothing)
    b, w = ([[int(m != f_mb[s] and rng.random() < 0.4 * density) for m in range(mbs)] for s in range(n)] for _ in range(2))
    # whether the first W unit, or a later one, is behind a B unit of its step on another stream
    through = [rng.choice([0, 1, 2]) if slot_of[1] != slot_of[2] and any(x and y for x, y in zip(b[s], w[s])) else 0 for s in range(n)]
    waits = plan(mbs, f_mb, b, w, through, slot_of)
    assert all(1 <= m < s for s, i, j, m in waits)
    # clock[i][j]: last step of slot j that slot i's stream is ordered behind; at_end[s][i]: the same when step s was marked
    clock, at_end = [[0] * 3 for _ in range(3)], {0: [[0] * 3 for _ in range(3)]}
    latest = {}                      # (kind, microbatch): last step before this one with such work

    def behind(i, j, step, of):
        clock[i] = [max(a, c) for a, c in zip(clock[i], of)]
        clock[i][j] = max(clock[i][j], step)

    def take(s, i):
        for _, _, j, m in [x for x in waits if x[:2] == (s, i)]:
            assert clock[i][j] < m, f"step {s}: slot {i} waits again for step {m} of slot {j}"
            behind(i, j, m, at_end[m][j])

    for s in range(1, n + 1):
        own_w = slot_of[2] == 2 and any(w[s - 1])
        for i in range(3):
            if slot_of[i] != i:
                continue
            if i == 2 and own_w and through[s - 1] == 1:
                behind(2, slot_of[1], s - 1, clock[slot_of[1]])
            take(s, i)
        # the hazards, from the data alone: F writes a microbatch's stash, B reads it and adds to it, W reads both
        work = [(0, f_mb[s - 1])] if f_mb[s - 1] >= 0 else []
        work += [(1, m) for m in range(mbs) if b[s - 1][m]] + [(2, m) for m in range(mbs) if w[s - 1][m]]
        for kind, m in work:
            for other in {0: (1, 2), 1: (0, 2), 2: (0, 1)}[kind]:
                i, j, step = slot_of[kind], slot_of[other], latest.get((other, m), 0)
                assert i == j or clock[i][j] >= step, f"step {s}: {'FBW'[kind]}({m}) is not behind {'FBW'[other]}({m}) of step {step}"
        # and every stream, with work or without, behind the whole of the step before last
        for i in set(slot_of):
            for j in set(slot_of):
                assert i == j or clock[i][j] >= s - 2, f"step {s}: slot {i} is not behind step {s - 2} of slot {j}"
        if any(w[s - 1]) and (through[s - 1] == 2 or (through[s - 1] == 1 and not own_w)):      # (a shared slot waits in the middle of its step)
            behind(slot_of[2], slot_of[1], s - 1, clock[slot_of[1]])
        at_end[s] = [list(c) for c in clock]
        for key in work:
            latest[key] = s
