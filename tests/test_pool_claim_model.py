"""Step-interleaved model of the claims of fresh frames from a pool's bump word:
one load, then an add while the load left a margin, else compare-and-swap; an
add that passes the pool's end puts the word back.

Each claimer is a generator that performs one access to the shared word per
step; a seeded scheduler picks who takes the next step.  The pool and the margin
are so small that several adds pass the end at once.  No frame may be handed
out twice or beyond the pool, the word must end at the number of frames handed
out, and a claim may fail only when, at some moment of it, the pool had fewer
frames left than it asked for.  A pool that every claimer fits into refuses
none.  Taking failed adds back by subtraction must be caught."""
import random

import pytest


class Pool:
    def __init__(self, size, take_back):
        self.size, self.word, self.take_back = size, 0, take_back
        self.owned = set()
        self.top = 0  # frames handed out

    def grant(self, base, n):
        frames = set(range(base, base + n))
        assert base + n <= self.size and not frames & self.owned, "a frame handed out twice or beyond the pool"
        self.owned |= frames
        self.top += n


def claim(pool, n, margin, out):
    short = [False]  # whether the pool was too full for this claim at one of its steps

    def look():
        short[0] |= pool.top + n > pool.size

    cur = pool.word
    look()
    yield
    if cur + n + margin <= pool.size:
        cur = pool.word
        pool.word += n
        look()
        if cur + n <= pool.size:
            pool.grant(cur, n)
            out.append(n)
            yield
            return
        yield
        if pool.take_back == "subtract":
            cur = pool.word - n
            pool.word = cur
            yield
        elif cur <= pool.size:
            pool.word = cur
            yield
    while cur + n <= pool.size or cur > pool.size:
        look()
        if cur > pool.size:
            cur = pool.word
        elif pool.word == cur:
            pool.word = cur + n
            pool.grant(cur, n)
            out.append(n)
            yield
            return
        else:
            cur = pool.word
        yield
    look()
    assert short[0], "a claim refused while the pool had room"


def claimer(pool, sizes, margin, out):
    for n in sizes:
        yield from claim(pool, n, margin, out)


def run(seed, take_back="exchange", fits=False):
    rng = random.Random(seed)
    sizes = [[rng.randint(1, 9) for _ in range(rng.randint(1, 4))] for _ in range(rng.randint(2, 6))]
    total = sum(map(sum, sizes))
    pool = Pool(total if fits else rng.randint(1, max(1, total)), take_back)
    out = []
    live = [claimer(pool, s, rng.randint(0, 3), out) for s in sizes]
    for _ in range(20000):
        if not live:
            break
        a = rng.choice(live)
        try:
            next(a)
        except StopIteration:
            live.remove(a)
    assert not live, "a claim that does not end"
    assert pool.word == pool.top == sum(out) <= pool.size
    if fits:
        assert pool.top == total


@pytest.mark.parametrize("fits", [False, True])
def test_claims_are_exact(fits):
    for seed in range(4000):
        run(seed, fits=fits)


def test_subtracting_failed_adds_is_caught():
    caught = 0
    for seed in range(4000):
        try:
            run(seed, take_back="subtract")
        except AssertionError:
            caught += 1
    assert caught > 0
