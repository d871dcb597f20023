"""The clause phase's step numbers when every wave starts with a pair of its own.

Of T steps in pairs (2j, 2j + 1), wave w of W starts a sweep with pair w; the
pairs from W on come from a counter that runs on across an item's sweeps, of
which a sweep consumes floor(T/2) numbers.  Modelled on the host for random
interleavings of the waves."""
import random

import pytest


def run_sweep(T, W, counter, base, rng):
    taken = []
    state = [2 * w for w in range(W)]
    live = [w for w in range(W) if state[w] < T]
    while live:
        w = rng.choice(live)
        taken.append(state[w])
        if state[w] % 2 == 0:
            state[w] += 1
        else:
            state[w] = 2 * (W + counter[0] - base)
            counter[0] += 1
        if state[w] >= T:
            live.remove(w)
    return taken


@pytest.mark.parametrize("T,W", [(1, 1), (1, 16), (2, 1), (3, 2), (28, 16), (31, 16), (32, 16), (33, 16), (191, 8),
                                 (192, 16)])
def test_every_step_once_and_numbers_per_sweep(T, W):
    rng = random.Random(T * 100 + W)
    for _ in range(20):
        counter = [0]
        for s in range(6):
            assert sorted(run_sweep(T, W, counter, s * (T // 2), rng)) == list(range(T))
            assert counter[0] == (s + 1) * (T // 2)


def test_no_steps():
    """A split member without records: nothing taken, no number consumed."""
    counter = [0]
    for s in range(3):
        assert run_sweep(0, 16, counter, 0, random.Random(s)) == []
    assert counter == [0]


@pytest.mark.parametrize("T,W", [(28, 4), (31, 4), (33, 16), (40, 16)])
@pytest.mark.parametrize("off", [-1, 1])
def test_another_count_per_sweep_is_caught(T, W, off):
    """One number more or less a sweep repeats or skips steps from the second on
    (where the counter hands out any)."""
    counter, rng = [0], random.Random(T)
    right = []
    for s in range(4):
        try:
            right.append(sorted(run_sweep(T, W, counter, s * (T // 2 + off), rng)) == list(range(T)))
        except IndexError:
            right.append(False)
    assert right[0] and not all(right[1:])
