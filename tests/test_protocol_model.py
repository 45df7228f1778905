"""Host-side model of the inter-workgroup protocols of the one-pass encoders: the range
words that workgroups exchange through the workspace, the waits on them, and the rule by
which the workspace is left all zero without a clearing pass.  Each wave is a coroutine
that yields at every access to the shared words; a seeded scheduler interleaves the waves
of all workgroups at random.  Checked on thousands of schedules: no wave ever waits for
a word that has already been cleared (that would hang the kernel), every wave sees all
words of its chunk, and every word and counter is zero at the end.

The model restates the protocol, it shares nothing with the kernels:
  rotated kernels   per item: [workgroup barrier] publish, wait for all words of the chunk,
                    clear the own word of the workgroup's PREVIOUS chunk
  one word per workgroup (more than 16 workers): wave 0 publishes behind the barrier and clears
  one reader (more than 32 workers): the same, and wave 0 alone polls; it hands the result to the other
                    waves through the cell in which it gathered the workgroup's own maximum
  spread workers    (small chunks of more workers than a workgroup holds) one reader, and an item has several chunks: a
                    word per workgroup and chunk, published, waited for and cleared together, fewer in the last item;
                    the words that were read are handed over in a table of their own
  pipelined kernel  (unrotated bf16) no barriers: publish item k + 1, wait for item k,
                    clear the own word of item k - 2
  both              the workgroups of a chunk count themselves off for a workgroup's last
                    chunk(s); the last one clears all of the chunk's words and the counter
and deliberately wrong variants (the pipelined kernel clearing item k - 1, the one reader without a barrier
in front of the hand-over or in front of the cell's next use, the spread workers without one of their two barriers,
clearing the words of the current item, or as many of the last item as of the one before it) must be caught.  With a bound on the polls of a
wait every wave still ends, and the waves of a workgroup go on with one and the same result.
"""
import random

import pytest


class Hang(Exception):
    pass


class World:
    def __init__(self, W, V, chunks, words_per_workgroup=None):
        self.W, self.V = W, V
        self.P = words_per_workgroup or V     # publishing waves per workgroup
        self.word = {(c, w, v): 0 for c in range(chunks) for w in range(W) for v in range(self.P)}
        self.done = [0] * chunks
        self.expired = False      # a wait has given up
        self.seen = {}            # (w, v, c) -> the words a wave saw when its wait ended

    def all_words(self, c):
        return [self.word[(c, w, v)] for w in range(self.W) for v in range(self.P)]


class Barrier:
    def __init__(self, parties):
        self.parties, self.count, self.generation = parties, 0, 0


def _barrier(bar):
    gen = bar.generation
    bar.count += 1
    if bar.count == bar.parties:
        bar.count = 0
        bar.generation += 1
    while bar.generation == gen:
        yield "barrier"


def _wait(world, c, me):
    while True:
        yield "poll"
        words = world.all_words(c)
        if all(x != 0 for x in words):
            world.seen[me + (c,)] = words
            return


def _count_off(world, c):
    yield "atomic"
    arrived = world.done[c]
    world.done[c] += 1
    if arrived == world.W - 1:
        for w in range(world.W):
            for v in range(world.P):
                yield "clear"
                world.word[(c, w, v)] = 0
        world.done[c] = 0


def rotated_wave(world, bar, w, v, items):
    """One word per wave; a workgroup barrier (the rotation's exchanges) in front of every publication."""
    prev = None
    for c in items:
        yield from _barrier(bar)
        yield "publish"
        world.word[(c, w, v)] = 100 + c
        yield from _wait(world, c, (w, v))
        if prev is not None:
            yield "clear"
            world.word[(prev, w, v)] = 0
        prev = c
    yield from _barrier(bar)
    if v == 0 and prev is not None:
        yield from _count_off(world, prev)


def workgroup_word_wave(world, bar, w, v, items):
    """One word per WORKGROUP (more than 16 workers): wave 0 publishes behind the barrier and
    clears; every wave polls."""
    prev = None
    for c in items:
        yield from _barrier(bar)
        if v == 0:
            yield "publish"
            world.word[(c, w, 0)] = 100 + c
        yield from _wait(world, c, (w, v))
        if v == 0 and prev is not None:
            yield "clear"
            world.word[(prev, w, 0)] = 0
        prev = c
    yield from _barrier(bar)
    if v == 0 and prev is not None:
        yield from _count_off(world, prev)


def one_reader_wave(world, bar, w, v, items, limit=None, handover_barrier=True, rotation_barrier=True):
    """One word per workgroup, read by wave 0 for all.  bar.cell: a place per wave for its maximum; the first one
    then carries the result of the wait.  limit: polls after which the wait gives up."""
    if not hasattr(bar, "cell"):
        bar.cell, bar.results = [0] * bar.parties, {}
    prev = None
    for c in items:
        if rotation_barrier:
            yield from _barrier(bar)      # the rotation's exchange
        yield "maximum"
        bar.cell[v] = 100 + c
        yield from _barrier(bar)
        if v == 0:
            assert bar.cell == [100 + c] * bar.parties, "a maximum was overwritten before it was gathered"
            yield "publish"
            world.word[(c, w, 0)] = 100 + c
        yield from _barrier(bar)          # the last exchange
        if v == 0:
            polls, done = 0, False
            while not done and (limit is None or polls <= limit):
                yield "poll"
                words = world.all_words(c)
                done = all(x != 0 for x in words)
                polls += 1
            if not done:
                world.expired = True
            elif prev is not None:
                yield "clear"
                world.word[(prev, w, 0)] = 0
            yield "hand over"
            bar.cell[0] = ("result", c, tuple(words))
        if handover_barrier:
            yield from _barrier(bar)
        yield "take over"
        got = bar.cell[0]
        assert got[:2] == ("result", c) if isinstance(got, tuple) else False, "a wave took something else over"
        assert bar.results.setdefault(c, got) == got
        world.seen[(w, v, c)] = list(got[2])
        prev = c
    yield from _barrier(bar)
    if v == 0 and prev is not None:
        yield from _count_off(world, prev)


def spread_wave(world, bar, w, v, items, per_item=1, limit=None, gather_barrier=True, handover_barrier=True,
                clear_current=False, clear_as_before=False):
    """An item is per_item consecutive chunks, the last one what is left of them.  bar.cell: a place per wave for its
    maximum; bar.got: the words that wave 0 has read."""
    if not hasattr(bar, "cell"):
        bar.cell, bar.got, bar.results = [0] * bar.parties, None, {}
    prev = []
    for c in items:
        chunks = [p for p in range(c * per_item, (c + 1) * per_item) if p < len(world.done)]
        yield "maximum"
        bar.cell[v] = 100 + c
        if gather_barrier:
            yield from _barrier(bar)
        if v == 0:
            for p in chunks:
                assert bar.cell == [100 + c] * bar.parties, "a maximum is missing or was overwritten"
                yield "publish"
                world.word[(p, w, 0)] = 100 + c
            polls, done = 0, False
            while not done and (limit is None or polls <= limit):
                yield "poll"
                words = []
                for p in chunks:
                    words += world.all_words(p)
                    yield "read"                      # (the words are read one after the other)
                done = all(x != 0 for x in words)
                polls += 1
            bar.got = (c, tuple(words))
            if not done:
                world.expired = True
            else:
                for p in chunks if clear_current else prev[:len(chunks)] if clear_as_before else prev:
                    yield "clear"
                    world.word[(p, w, 0)] = 0
        if handover_barrier:
            yield from _barrier(bar)
        yield "take over"
        assert bar.got is not None and bar.got[0] == c, "a wave took something else over"
        assert bar.results.setdefault(c, bar.got) == bar.got
        for k, p in enumerate(chunks):
            world.seen[(w, v, p)] = [x - c + p if x else 0 for x in bar.got[1][k * world.W:(k + 1) * world.W]]
        prev = chunks
    if v == 0 and prev:
        yield "atomic"
        arrived = world.done[prev[0]]
        world.done[prev[0]] += 1
        if arrived == world.W - 1:
            for p in prev:
                for u in range(world.W):
                    yield "clear"
                    world.word[(p, u, 0)] = 0
            world.done[prev[0]] = 0


def pipelined_wave(world, bar, w, v, items, clear_lag=2):
    """No barrier between items: the range of item k + 1 is published before the wait for item k."""
    if not items:
        return
    yield "publish"
    world.word[(items[0], w, v)] = 100 + items[0]
    for k, c in enumerate(items):
        if k + 1 < len(items):
            yield "publish"
            world.word[(items[k + 1], w, v)] = 100 + items[k + 1]
        yield from _wait(world, c, (w, v))
        if k >= clear_lag:
            yield "clear"
            world.word[(items[k - clear_lag], w, v)] = 0
    yield from _barrier(bar)
    if v == 0:
        for c in items[-clear_lag:]:
            yield from _count_off(world, c)


def run(kind, W, V, groups, rounds, seed, words_per_workgroup=None, missing=0, **kw):
    """groups peer groups of W workgroups; group q handles items q, q + groups, ...  An item is a chunk, or
    per_item of them (missing: fewer in the last item)."""
    rng = random.Random(seed)
    items_in_all = groups * rounds
    chunks = items_in_all * kw.get("per_item", 1) - missing
    world = World(W, V, chunks, words_per_workgroup)
    waves = []
    for q in range(groups):
        items = list(range(q, items_in_all, groups))
        for w in range(W):
            bar = Barrier(V)
            for v in range(V):
                waves.append(kind(world, bar, w, v, items, **kw))
    idle = 0
    while waves:
        i = rng.randrange(len(waves))
        before = (dict(world.word), list(world.done))
        try:
            step = next(waves[i])
        except StopIteration:
            waves.pop(i)
            idle = 0
            continue
        if step in ("poll", "read", "barrier") and before == (world.word, world.done):
            idle += 1
            if idle > 2000 * len(waves):
                raise Hang(f"no progress: {len(waves)} waves stuck")
        else:
            idle = 0
    assert len(world.seen) == chunks * W * V
    if world.expired:             # (the workspace then has to be cleared, and maxima may be missing)
        assert all(x in (0, 100 + c) for (w, v, c), words in world.seen.items() for x in words)
        return world
    assert all(x == 0 for x in world.word.values()), "a range word is left set"
    assert all(x == 0 for x in world.done), "a counter is left set"
    for (w, v, c), words in world.seen.items():
        assert all(x == 100 + c for x in words), "a wave saw a word of another chunk"
    return world


@pytest.mark.parametrize("W,V,groups,rounds", [(2, 2, 1, 1), (2, 2, 1, 4), (3, 2, 2, 3), (2, 3, 1, 5), (4, 1, 2, 4)])
def test_rotated_protocol_clears_itself_and_never_hangs(W, V, groups, rounds):
    for seed in range(300):
        run(rotated_wave, W, V, groups, rounds, seed)


@pytest.mark.parametrize("W,V,groups,rounds", [(2, 2, 1, 1), (2, 3, 1, 4), (3, 2, 2, 3), (5, 2, 1, 4)])
def test_workgroup_word_protocol_clears_itself_and_never_hangs(W, V, groups, rounds):
    for seed in range(300):
        run(workgroup_word_wave, W, V, groups, rounds, seed, words_per_workgroup=1)


@pytest.mark.parametrize("W,V,groups,rounds", [(2, 2, 1, 1), (2, 3, 1, 4), (3, 2, 2, 3), (5, 2, 1, 4)])
def test_one_reader_protocol_clears_itself_and_never_hangs(W, V, groups, rounds):
    for seed in range(300):
        assert not run(one_reader_wave, W, V, groups, rounds, seed, words_per_workgroup=1).expired


@pytest.mark.parametrize("limit", [0, 3])
@pytest.mark.parametrize("W,V,groups,rounds", [(2, 2, 1, 1), (2, 3, 1, 4), (3, 2, 2, 3)])
def test_one_reader_that_gives_up_ends_with_one_result_per_workgroup(W, V, groups, rounds, limit):
    expired = sum(run(one_reader_wave, W, V, groups, rounds, seed, words_per_workgroup=1, limit=limit).expired
                  for seed in range(300))
    assert expired > 0


@pytest.mark.parametrize("parts,V,groups,rounds,per_item,missing", [
    (2, 2, 1, 1, 1, 0), (2, 2, 1, 4, 3, 2), (3, 2, 2, 3, 2, 1), (3, 1, 1, 5, 4, 0), (2, 3, 2, 2, 3, 1)])
def test_spread_protocol_clears_itself_and_never_hangs(parts, V, groups, rounds, per_item, missing):
    for seed in range(300):
        assert not run(spread_wave, parts, V, groups, rounds, seed, words_per_workgroup=1, per_item=per_item,
                       missing=missing).expired


@pytest.mark.parametrize("limit", [0, 2])
def test_spread_reader_that_gives_up_ends_with_one_result_per_workgroup(limit):
    expired = sum(run(spread_wave, 2, 3, 1, 4, seed, words_per_workgroup=1, per_item=3, missing=1, limit=limit).expired
                  for seed in range(300))
    assert expired > 0


@pytest.mark.parametrize("wrong", [dict(gather_barrier=False), dict(handover_barrier=False), dict(clear_current=True),
                                   dict(clear_as_before=True)])
def test_the_model_catches_a_wrong_spread_protocol(wrong):
    def catches(seed):
        try:
            run(spread_wave, 2, 3, 1, 4, seed, words_per_workgroup=1, per_item=3, missing=2, **wrong)
        except (Hang, AssertionError):
            return True
        return False
    assert any(catches(seed) for seed in range(300))


@pytest.mark.parametrize("without", ["handover_barrier", "rotation_barrier"])
def test_the_model_catches_a_missing_barrier_around_the_hand_over(without):
    caught = 0
    for seed in range(300):
        try:
            run(one_reader_wave, 2, 3, 1, 5, seed, words_per_workgroup=1, **{without: False})
        except (Hang, AssertionError):
            caught += 1
    assert caught > 0


@pytest.mark.parametrize("W,V,groups,rounds", [(2, 2, 1, 1), (2, 2, 1, 2), (2, 2, 1, 3), (3, 2, 2, 4), (2, 3, 1, 6), (4, 1, 2, 5)])
def test_pipelined_protocol_clears_itself_and_never_hangs(W, V, groups, rounds):
    for seed in range(300):
        run(pipelined_wave, W, V, groups, rounds, seed)


def test_the_model_catches_a_word_cleared_one_item_too_early():
    """Clearing the own word of item k - 1 after the wait for item k is wrong for the
    pipelined kernel (a peer may still be waiting for item k - 1): some schedule hangs."""
    caught = 0
    for seed in range(300):
        try:
            run(pipelined_wave, 2, 2, 1, 5, seed, clear_lag=1)
        except (Hang, AssertionError):
            caught += 1
    assert caught > 0
