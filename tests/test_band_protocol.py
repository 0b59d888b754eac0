"""A CPU model of how the bands of one matrix hand their rows on (sw_bands.h): tagged words that are overwritten in
place, read 32 columns at a time and asked for in the middle of the batch before, by as many waves as happen to run.
Any order in which the waves take their steps must give every band the row above it, and end."""
import random

import pytest

BATCH, LANES = 32, 64


class Wave:
    """One wave of the sweep: takes bands from the counter in order until none is left.  step() makes its next access to
    shared memory (a pull, a read of a batch, or the store of one step) and returns False when it has ended."""

    def __init__(self, world):
        self.w = world
        self.program = self.run()
        self.waiting = False

    def step(self):
        return next(self.program, False)

    def words(self, c, tag):
        """What the lanes' loads of batch c return: (value, tag) per column; past the subject the tag alone."""
        w = self.w
        out = []
        for j in range(BATCH * c, BATCH * c + BATCH):
            out.append(w.row[j] if tag and j < w.n else (None, tag))
        return out

    def run(self):
        w = self.w
        steps = -(-(w.n + LANES - 1) // BATCH) * BATCH
        while True:
            band = w.counter
            w.counter += 1
            yield True
            if band >= w.bands:
                return
            tag, last = band, band == w.bands - 1
            v = self.words(0, tag)
            yield True
            for c in range(steps // BATCH):
                while any(t != tag for _, t in v):
                    self.waiting = True
                    yield True
                    v = self.words(c, tag)
                self.waiting = False
                for j, (value, _) in enumerate(v):
                    if tag and BATCH * c + j < w.n and value != (band - 1, BATCH * c + j):
                        raise AssertionError(f"band {band} read {value} for column {BATCH * c + j}")
                nxt = None
                for u in range(BATCH):
                    if u == w.ask:
                        nxt = self.words(c + 1, tag)
                        yield True
                    j = BATCH * c + u - w.skew             # lane 63's column
                    if not last and 0 <= j < w.n:
                        w.row[j] = ((band, j), w.hand_on(tag))
                        yield True
                v = nxt
            w.done += 1


class World:
    def __init__(self, n, bands, waves, ask, hand_on=lambda tag: tag + 1, skew=LANES - 1):
        self.n, self.bands, self.ask, self.hand_on, self.skew = n, bands, ask, hand_on, skew
        self.row = [(None, 0)] * n
        self.counter = self.done = 0
        self.waves = [Wave(self) for _ in range(waves)]

    def run(self, pick):
        running = list(self.waves)
        idle = 0
        while running:
            wave = pick(running)
            if not wave.step():
                running.remove(wave)
            # (no wave but waiting ones for long: nobody goes on any more)
            idle = idle + 1 if all(x.waiting for x in running) and running else 0
            if idle > 50 * len(self.waves) + 200:
                raise AssertionError("every wave waits")
        assert self.done == self.bands


def orders(rng):
    yield "random", lambda ws: rng.choice(ws)
    yield "first come", lambda ws: ws[0] if not ws[0].waiting else rng.choice(ws)
    yield "last come", lambda ws: ws[-1] if not ws[-1].waiting else rng.choice(ws)
    # a favoured wave runs ahead for long stretches
    state = {"w": None, "k": 0}

    def bursts(ws):
        if state["w"] not in ws or state["k"] <= 0 or state["w"].waiting:
            state["w"], state["k"] = rng.choice(ws), rng.randint(1, 400)
        state["k"] -= 1
        return state["w"]
    yield "bursts", bursts


@pytest.mark.parametrize("ask", [0, 16])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 96, 129, 200])
def test_every_order_hands_the_rows_on(n, ask):
    rng = random.Random(n * 100 + ask)
    for bands, waves in ((1, 1), (2, 2), (3, 1), (5, 2), (6, 6), (4, 9)):
        for name, pick in orders(rng):
            World(n, bands, waves, ask).run(pick)


@pytest.mark.parametrize("ask", [0, 16])
def test_planted_mistakes_show(ask):
    def fails(**kw):
        seen = 0
        for seed in range(6):
            rng = random.Random(seed)
            for _, pick in orders(rng):
                try:
                    World(200, 5, 3, ask, **kw).run(pick)
                except AssertionError:
                    seen += 1
        return seen
    assert fails() == 0
    # a band that tags its row as its own (the band below never sees it), or with the number two below
    assert fails(hand_on=lambda tag: tag) > 0
    assert fails(hand_on=lambda tag: tag + 2) > 0
    # a store ahead of the column that was read: it overwrites words of later batches
    assert fails(skew=-BATCH) > 0
