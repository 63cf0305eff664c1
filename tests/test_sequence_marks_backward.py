"""The exchange of the whole-sequence backward kernel (csrc/lstm_xcd.hip), as a model on the CPU: who may still read a word of a message
when it is marked for its next use, and who may still be about to mark it when it is written.

Members stand in squares of four.  A member has four waves; wave w < S owns one group of eight units, if it exists.  A step of a wave:
load the partial sums of its units, one from every square, until no word is marked (not in step 0); wait for its own stores; send dz of
its units; put the marks back on the sums it has read and mark its own words of the dz block of two steps ago; load dz of the square's
member w until no word is marked; barrier; send the partial sums of every fourth tile (two groups of units) of the member's quarter.
In fp32 sums that are not finite are taken again first, tile by tile, from the dz of the whole square as it lies in memory.  (There another
barrier follows, for the sums in LDS; the messages do without.)  Blocks of both kinds are four that take turns.  A wave's stores arrive in any order, those to one word in order, at the
latest at its next wait.  A member without units and without tiles takes no part."""
import random

import pytest

BLOCKS = 4


class Broken(Exception):
    pass


def walk(groups, S, steps, rng, back, wait, again=False):
    """One run under a random schedule.  back: of how many steps ago the dz block is that is marked; wait: whether marks are waited for;
    again: whether some sums are taken again."""
    real = (groups + S - 1) // S
    members = (real + 3) // 4 * 4
    tiles = (groups + 1) // 2
    quarter = (tiles + 3) // 4
    squares = members // 4
    dz = [[None] * groups for _ in range(BLOCKS)]                  # the step whose values a word holds; None: marked
    sums = [[[None] * groups for _ in range(squares)] for _ in range(BLOCKS)]
    arrived = [0] * members

    def wave(m, w):
        unit = m * S + w if w < S and m * S + w < groups else None
        square, first = m // 4, m % 4 * quarter
        whole = [g for g in range(4 * square * S, 4 * (square + 1) * S) if g < groups]
        mine = [t for t in range(first, min(first + quarter, tiles)) if (t - first) % 4 == w]
        peer = [g for g in range((4 * square + w) * S, (4 * square + w + 1) * S) if g < groups]
        if m * S >= groups and first >= tiles:
            return
        pending = []

        def drain(everything):
            while pending and (everything or rng.random() < 0.5):
                at = rng.randrange(len(pending))
                at = next(i for i, p in enumerate(pending) if p[0] is pending[at][0] and p[1] == pending[at][1])
                row, i, value = pending.pop(at)
                row[i] = value

        def barrier():
            arrived[m] += 1
            full = (arrived[m] + 3) // 4 * 4
            while arrived[m] < full:
                drain(False)
                yield False

        for step in range(steps):
            if w < S:
                if step > 0 and unit is not None:
                    while True:
                        seen = [sums[step % BLOCKS][sq][unit] for sq in range(squares)]
                        if None not in seen:
                            break
                        drain(False)
                        yield False
                    if any(v != step for v in seen):
                        raise Broken("step %d read sums of another step" % step)
                if wait:
                    drain(True)
                if unit is not None and step + 1 < steps:
                    pending.append((dz[step % BLOCKS], unit, step))
                drain(False)
                yield True
                if unit is not None and step > 0:
                    for sq in range(squares):
                        pending.append((sums[step % BLOCKS][sq], unit, None))
                    pending.append((dz[(step - back) % BLOCKS], unit, None))
                yield True
            if step + 1 == steps:
                drain(True)
                return
            while True:
                seen = [dz[step % BLOCKS][g] for g in peer]
                if None not in seen:
                    break
                drain(False)
                yield False
            if any(v != step for v in seen):
                raise Broken("step %d read dz of another step" % step)
            yield from barrier()
            redo = again and rng.random() < 0.5
            for t in mine:
                for g in whole if redo else ():
                    if dz[step % BLOCKS][g] != step:
                        raise Broken("step %d multiplied again dz of another step" % step)
                    if rng.random() < 0.2:
                        drain(False)
                        yield True
                for g in (2 * t, 2 * t + 1):
                    if g < groups:
                        pending.append((sums[(step + 1) % BLOCKS][square], g, step + 1))
            drain(False)
            yield True

    waves = [(m, wave(m, w)) for m in range(members) for w in range(4)]
    slow = {rng.randrange(members) for _ in range(rng.choice((1, 1, 3)))}
    idle = 0
    while waves:
        i = rng.randrange(len(waves))
        if waves[i][0] in slow and rng.random() < 0.95:
            continue
        try:
            idle = 0 if next(waves[i][1]) else idle + 1
        except StopIteration:
            waves.pop(i)
            idle = 0
        if idle > 600 * (len(waves) + 1):
            raise Broken("everybody waits")


SIZES = ((2, 1), (4, 1), (6, 1), (10, 1), (12, 1), (32, 1), (36, 2), (38, 2), (68, 3), (84, 3))      # groups of eight units, S


def outcomes(seeds, back=2, wait=True, again=False):
    bad = 0
    for seed in range(seeds):
        rng = random.Random(seed)
        groups, S = SIZES[seed % len(SIZES)]
        try:
            walk(groups, S, 11, rng, back, wait, again)
        except Broken:
            bad += 1
    return bad


def test_no_word_is_marked_or_written_too_early():
    assert outcomes(60) == 0


def test_sums_taken_again_find_the_dz_they_were_made_of():
    assert outcomes(60, again=True) == 0
    assert outcomes(40, back=1, again=True) > 0


def test_the_model_sees_marks_too_early_and_marks_not_waited_for():
    assert outcomes(40, back=1) > 0
    assert outcomes(40, wait=False) > 0
