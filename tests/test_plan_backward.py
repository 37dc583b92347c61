"""The work split of the 16-bit backward on the host (CPU only): the choice is the best one by the stated model, and
choosing it stays cheap for long packed batches, whose layout is new in every iteration."""
import heapq
import time

import numpy as np
import pytest

from plan_lib import backward_split

STEP_US, UNIT_US, EMPTY_US, TILE_US, DIAG_US, Q_US = 1.9, 13.0, 1.0, 5.0, 1.7, 8.0


def layout(rng, tokens, lo, hi):
    cu = [0]
    while cu[-1] < tokens:
        cu.append(min(tokens, cu[-1] + int(rng.integers(lo, hi + 1))))
    return np.array(cu, dtype=np.int32)


def first_xcd(hkv, n_units):
    """unit numbers of the first XCD in launch order"""
    if hkv % 8 == 0:
        return [u for u in range(n_units) for _ in range(hkv // 8)]
    if 8 % hkv == 0:
        return range(0, n_units, 8 // hkv)
    return [i // hkv for i in range(0, n_units * hkv, 8)]


def model(cu, hq, hkv, d, b, n, cb, ns, n_cu=256):
    """When the last compute unit of an XCD ends, with the units listed one by one."""
    T, G = int(cu[-1]), hq // hkv
    scale = 0.6 if d == 64 else 1.0
    start_of = lambda i: int(cu[np.searchsorted(cu, i, side="right") - 1])
    end_of = lambda i: int(cu[np.searchsorted(cu, i, side="right")])
    steps = []
    for ch in range(-(-T // (cb * 32))):
        for t in range(min(-(-T // 128), (ch + 1) * cb // 4)):
            last = min((end_of(min(t * 128 + 127, T - 1)) - 1) // 32, (ch + 1) * cb - 1)
            steps.append((max(0, last - max(t * 4, ch * cb) + 1) + 1) // 2)
    jobs = []
    for u in first_xcd(hkv, len(steps) * ns):
        sp, s = u // len(steps), steps[u % len(steps)]
        jobs.append((n * G - sp + ns - 1) // ns * s * STEP_US * scale + UNIT_US if s else EMPTY_US)
    tiles = -(-T // 256)
    for u in first_xcd(hkv, tiles * n * G):
        t = tiles - 1 - u // (n * G)
        keys = min(t * 256 + 255, T - 1) // 128 - start_of(t * 256) // 128 + 1
        jobs.append(Q_US + keys * TILE_US * scale + (b + u // G % n) * DIAG_US * scale)
    free = [0.0] * (n_cu // 8)
    for us in jobs:
        heapq.heapreplace(free, free[0] + us)
    return max(free)


@pytest.mark.parametrize("tokens,lo,hi,hq,hkv,d,b,n", [
    (1, 1, 1, 2, 2, 128, 0, 7), (700, 1, 90, 8, 2, 64, 0, 4), (2048, 2048, 2048, 32, 8, 128, 6, 1), (1500, 0, 700, 6, 3, 128, 1, 2),
    (3000, 100, 900, 32, 16, 128, 0, 1), (4096, 4096, 4096, 32, 8, 128, 0, 7), (2500, 2500, 2500, 10, 5, 64, 2, 3),
    (5000, 256, 4096, 64, 4, 128, 3, 1), (4000, 4000, 4000, 1, 1, 128, 0, 1),
])
def test_the_choice_is_the_best_by_the_model(tokens, lo, hi, hq, hkv, d, b, n):
    cu = layout(np.random.default_rng(tokens), tokens, lo, hi)
    cb, ns = backward_split(cu, hq, hkv, d, b, n)
    n_jh = n * (hq // hkv)
    options = {(c, s): model(cu, hq, hkv, d, b, n, c, s) for c in (8, 16, 32, 64, 128) for s in (1, 2, 3, 4, 6, 8)
               if s <= n_jh and (c <= 32 or n_jh <= 8) and (c == 8 or c * 16 < tokens)}
    # sums of at most a few hundred fp32 terms on the library's side
    assert options[cb, ns] <= min(options.values()) * (1 + 1e-4), (cb, ns, options)


def test_planning_time_grows_no_faster_than_the_tokens():
    """Seven calls of one step on a layout not seen before, 32/8 heads: 32 times the tokens may take 32 times as long."""
    rng = np.random.default_rng(7)
    best = {}
    for tokens in (16384, 524288):
        for _ in range(5):
            cu = layout(rng, tokens, 256, 4096)
            t0 = time.perf_counter()
            for j in range(6, -1, -1):
                backward_split(cu, 32, 8, 128, j, 1)
            best[tokens] = min(best.get(tokens, 1e9), time.perf_counter() - t0)
    assert best[524288] <= 32 * best[16384], best
