"""The exchange of the fp32 whole-sequence forward kernel (csrc/lstm_xcd.hip), as a model on the CPU: who may still read a block of h
when its next use is marked.

A member has four waves; wave w < S makes 8 of its 8 S units, and wave w reads every fourth 32 units of h_t, of all members.  A step of
a wave: load its part of block t until no word is marked; wait for its own stores; barrier; add up, which where a sum is not finite
reads the whole block again, word by word; send h_{t+1}; barrier.  Step t marks the words of block t + 3, one of four that take
turns.  A wave's stores arrive in any order, those to one word in order, at the latest at its next wait."""
import random

import pytest

BLOCKS, AHEAD = 4, 3


class Broken(Exception):
    pass


def walk(members, S, steps, rng, behind_barrier, retake):
    """One run under a random schedule.  retake: (member, wave) that read the block again in every step."""
    units = members * 8 * S
    block = [[-1] * units for _ in range(BLOCKS)]                # the step whose h it is; None: marked; -1: what lay in the workspace
    arrived = [[0] * 2 for _ in range(members)]                  # waves at each of the two barriers, ever

    def wave(m, w):
        own = range((m * S + w) * 8, (m * S + w) * 8 + 8) if w < S else range(0)
        mine = [u for u in range(units) if u // 32 % 4 == w]
        pending = []

        def store(t, value):
            pending.extend((t % BLOCKS, u, value) for u in own)

        def drain(everything):
            while pending and (everything or rng.random() < 0.5):
                at = rng.randrange(len(pending))
                first = next(i for i, p in enumerate(pending) if p[:2] == pending[at][:2])
                b, u, value = pending.pop(first)
                block[b][u] = value

        def barrier(which):
            arrived[m][which] += 1
            full = (arrived[m][which] + 3) // 4 * 4
            while arrived[m][which] < full:
                drain(False)
                yield False

        for t in range(AHEAD):
            store(t, None)
        drain(True)
        yield True
        store(0, 0)
        for t in range(steps):
            while True:
                seen = [block[t % BLOCKS][u] for u in mine]
                if None not in seen:
                    break
                drain(False)
                yield False
            if any(v != t for v in seen):
                raise Broken("step %d read h of another step" % t)
            drain(True)
            if not behind_barrier and t + AHEAD <= steps:
                store(t + AHEAD, None)
            yield True
            yield from barrier(0)
            if behind_barrier and t + AHEAD <= steps:
                store(t + AHEAD, None)
            if (m, w) in retake:
                for u in range(units):
                    if block[t % BLOCKS][u] != t:
                        raise Broken("a sum of step %d taken again read %r" % (t, block[t % BLOCKS][u]))
                    if u % 4 == 0:
                        yield True
            store(t + 1, t + 1)
            drain(False)
            yield True
            yield from barrier(1)

    waves = [(m, wave(m, w)) for m in range(members) for w in range(4)]
    for _, g in waves:                                           # all have marked their words before anybody begins
        next(g)
    slow = rng.randrange(members)
    idle = 0
    while waves:
        i = rng.randrange(len(waves))
        if waves[i][0] == slow and rng.random() < 0.9:
            continue
        try:
            idle = 0 if next(waves[i][1]) else idle + 1
        except StopIteration:
            waves.pop(i)
            idle = 0
        if idle > 400 * (len(waves) + 1):
            raise Broken("everybody waits")


def outcomes(behind_barrier, retakes):
    bad = 0
    for seed in range(30):
        rng = random.Random(seed)
        members, S = rng.choice(((3, 1), (5, 2), (6, 3), (9, 1)))
        retake = {(rng.randrange(members), rng.randrange(S))} if retakes else set()
        try:
            walk(members, S, 9, rng, behind_barrier, retake)
        except Broken:
            bad += 1
    return bad


@pytest.mark.parametrize("retakes", [False, True])
def test_blocks_are_marked_behind_the_barrier(retakes):
    assert outcomes(True, retakes) == 0


def test_marks_ahead_of_the_barrier_would_reach_readers():
    assert outcomes(False, True) > 0 and outcomes(False, False) > 0
