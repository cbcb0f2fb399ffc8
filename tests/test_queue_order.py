"""The order in which the persistent waves take work units (the loop of
csrc/esu.h, modelled here): whatever the number of units and waves, the grab
sizes, the split of the units over the queues and the interleaving of the
waves, every unit is taken exactly once."""

import random

import pytest

QUEUES = 8


def _taken(span, grid, grab, heavy_first, mix, begin, rng):
    end = begin + span
    heavy = [rng.random() < 0.5 for _ in range(span)]
    grabs = (min(4 * grab, 64), grab)
    heads = [[0] * QUEUES, [0] * QUEUES]
    taken = []
    tries = QUEUES - 1 if span // grid >= 16 or grid < 8 * QUEUES else 1

    def wave(w):
        home = w % QUEUES
        turn = w // QUEUES if tries < QUEUES - 1 else 0
        for sweep in range(0 if heavy_first else 1, 2):
            n = grabs[sweep]
            for t in range(tries + 1):
                x = home if t == 0 else (home + 1 + (turn + t - 1) % (QUEUES - 1)) % QUEUES
                lo = begin + x * n if mix else begin + span * x // QUEUES
                hi = end if mix else begin + span * (x + 1) // QUEUES
                while True:
                    idx = heads[sweep][x] * (QUEUES if mix else 1)
                    heads[sweep][x] += n
                    yield
                    if idx >= span or idx + lo >= hi:
                        break
                    idx += lo
                    taken.extend(u for u in range(idx, min(idx + n, hi))
                                 if not heavy_first or heavy[u - begin] == (sweep == 0))
                    yield

    waves = [wave(w) for w in range(grid)]
    while waves:
        i = rng.randrange(len(waves))
        if next(waves[i], True):
            waves[i] = waves[-1]
            waves.pop()
    return taken


@pytest.mark.parametrize("grid", [1, 2, 7, 8, 9, 63, 64, 65, 100])
@pytest.mark.parametrize("mix", [False, True])
def test_every_unit_once(grid, mix):
    rng = random.Random(grid * 2 + mix)
    for span in (0, 1, 7, 8, 9, 64, 65, 15 * grid, 16 * grid, 16 * grid + 1, rng.randint(0, 2500)):
        for grab in (1, 3, 16):
            begin = rng.choice([0, 5, 100])
            got = _taken(span, grid, grab, rng.random() < 0.5, mix, begin, rng)
            assert sorted(got) == list(range(begin, begin + span))
