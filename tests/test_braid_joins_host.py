"""The waits between braid steps: every order that a step needs follows from the waits that are made (directly or through other
streams' waits), and no wait is made that earlier ones imply."""
import ctypes as C
import random

import numpy as np
import pytest

import paper_2510_27257_amd as stp


def plan(has, last, through):
    f = stp.lib().stp_braid_plan_joins
    f.restype = C.c_int
    waits = np.zeros(1 << 14, np.int64)
    keep = [np.ascontiguousarray(a, np.uint8) for a in (has, last, through)]
    n = f(len(has), *(a.ctypes.data_as(C.c_void_p) for a in keep), waits.ctypes.data_as(C.c_void_p), len(waits))
    assert n >= 0
    return [(int(w) & 0xffff, int(w) >> 16 & 15, int(w) >> 20 & 15, int(w) >> 24) for w in waits[:n]]


@pytest.mark.parametrize("seed", range(40))
def test_waits_imply_every_needed_order_and_none_is_spare(seed):
    rng = random.Random(seed)
    n = 30
    density = rng.choice([0.3, 0.6, 1.0])
    has = [[int(rng.random() < density) for _ in range(3)] for _ in range(n)]
    last = [[int(rng.random() < 0.3) for _ in range(9)] for _ in range(n)]
    through = [int(h[1] and h[2] and rng.random() < 0.5) for h in has]
    waits = plan(has, last, through)
    assert all(1 <= m < s for s, i, j, m in waits)
    # clock[i][j]: last step of slot j that slot i's stream is ordered behind; at_end[s][i]: the same when step s was marked
    clock, at_end = [[0] * 3 for _ in range(3)], {0: [[0] * 3 for _ in range(3)]}

    def behind(i, j, step, of):
        clock[i] = [max(a, b) for a, b in zip(clock[i], of)]
        clock[i][j] = max(clock[i][j], step)

    for s in range(1, n + 1):
        for i in range(3):
            if i == 2 and through[s - 1]:
                behind(2, 1, s - 1, clock[1])
            for _, _, j, m in [w for w in waits if w[:2] == (s, i)]:
                assert clock[i][j] < m, f"step {s}: slot {i} waits again for step {m} of slot {j}"
                behind(i, j, m, at_end[m][j])
            for j in range(3):
                need = s - 1 if has[s - 1][i] and last[s - 1][3 * i + j] else s - 2      # without work too: the caller's own may follow
                assert j == i or clock[i][j] >= need, f"step {s}: slot {i} is not behind step {need} of slot {j}"
        at_end[s] = [list(c) for c in clock]
