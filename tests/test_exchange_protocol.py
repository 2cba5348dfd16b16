"""A CPU model of the batched kernel's exchange protocol (CPU only; the kernel
is in wr_batch.hip).

Heads and units of every group run the kernel's order of publishes and waits,
one read of one word per scheduling step, under random interleavings with
strongly skewed speeds.  A head is two agents, its waves that poll gate words
and publish y apart from each other, joined by the kernel's barriers; a unit is
one.  The words carry the kernel's tags:

* y slices, partial logits and gate words (with the e gate's context term)
  hold one parity bit of the step: a reader accepts a word whose bit matches
  and the model then checks that the word's full step is the one awaited (a
  parity match on another step is a misread);
* drawn samples sit in SS slots chosen by the step's tag modulo SS and carry
  16 bits of the tag.

A reader whose word was replaced before it was read waits forever (a lost
word, seen as a deadlock).

Both group modes are modelled.  Unit k's rows belong to the slice of head
k mod NH.  ALL (2 or 4 vectors per group): a head reads every gate word; its
publishing wave holds the head's own slice and polls that slice's words (3 unit
workgroups), its other waves the rest.  SLICE (8 vectors): every wave of a head
polls and publishes its part of the head's own slice, and the heads exchange
slices.  In both modes every head sums and draws every vector; one writer head
per vector's sample word.  `guard`: y_c is published only after a word of the step has come
from every unit of the group, so that none still has to read the y_c it
replaces: ALL behind the barrier that follows the gates (and after the partial
logits), SLICE once the publishing wave itself has seen a word of every unit.

The units wait for the drawn samples of step t - A of every lane of their
utterance: at the start of the step with a context lead A > 0 (before the
halves of h), after both halves with A = 0.  Sample words are published by idle
lanes too.

What the model leaves out: values, LDS staging, the split of one wave's poll
(its words are read one at a time, in order), memory-ordering effects of
the hardware (every write is visible to the next read), and the bounded waits'
clock.
"""
import random

import pytest


def run(mode="ALL", G=8, NH=2, L=2, B=16, F=4, A=1, rows=8, SS=None, seed=0, idle_publish=True, guard=True,
        max_ticks=4_000_000):
    rng = random.Random(seed)
    NU = 3 * NH
    if SS is None:
        SS = 2
        while SS < 2 * A + 2:
            SS *= 2
    V = G * L
    T = rows + (B - 1) * (F + 1 + A)
    mem = {}
    pos = lambda v, t: t - (v % B) * (F + 1 + A)
    act = lambda v, t: 0 <= pos(v, t) < rows

    def pub(key, tag):
        return ("w", key, tag)

    def wait1(key, tag):   # one parity-tagged word
        return ("r1", key, tag)

    def wait16(key, tag):  # a sample word: 16 bits of tag in its slot
        return ("r16", key, tag)

    def barrier(g, j, n):  # the n-th barrier of head j's two agents
        yield ("arrive", ("bar", g, j), 0)
        yield ("sync", ("bar", g, j), 2 * n)

    def samples(g, td):
        """The unit waits for the samples of step td of every lane of its utterance(s)."""
        if td < 0:
            return
        u0 = (g * L) // B
        nut = 1 if B >= L else L // B
        for vv in range(u0 * B, u0 * B + nut * B):
            if vv < V and (idle_publish or act(vv, td)):
                yield wait16(("S", vv // L, vv % L, (td + 1) % SS), td + 1)

    def head(g, j, p):
        """Agent p of head j: 0 the publishing wave (SLICE: the first wave), 1 the other waves."""
        n = 0
        own, rest = [k for k in range(NU) if k % NH == j], [k for k in range(NU) if k % NH != j]
        for s in range(T):
            tag = s + 1
            words = own if mode == "SLICE" or p == 0 else rest
            publishes = mode == "SLICE" or p == 0
            for k in words:
                yield wait1(("GATE", g, k), tag)
            # SLICE: without the guard the first wave's lanes alone poll every unit's first word
            if mode == "SLICE" and (guard or p == 0):
                for k in rest:
                    yield wait1(("GATE", g, k), tag)
            for half, out in (("YC", "PC"), ("YF", "PF")):
                late = guard and mode == "ALL" and half == "YC"    # behind the barrier
                if publishes and not late:
                    yield pub((half, g, j, p), tag)
                if mode == "SLICE":
                    for jj in range(NH):
                        for pp in range(2):
                            if jj != j:
                                yield wait1((half, g, jj, pp), tag)
                n += 1
                yield from barrier(g, j, n)
                if p == 0:
                    yield pub((out, g, j), tag)
                    if late:
                        yield pub((half, g, j, p), tag)
                    for jj in range(NH):
                        yield wait1((out, g, jj), tag)
                    if out == "PF":
                        for v in range(L):
                            if v % NH == j and (idle_publish or act(g * L + v, s)):
                                yield pub(("S", g, v, tag % SS), tag)
                n += 1
                yield from barrier(g, j, n)

    def unit(g, k):
        parts = (0, 1) if mode == "SLICE" else (0,)
        yield pub(("GATE", g, k), 1)
        for t in range(T - 1):
            tag = t + 1
            if A > 0:
                yield from samples(g, t - A)
            for half in ("YC", "YF"):
                for j in range(NH):
                    for p in parts:
                        yield wait1((half, g, j, p), tag)
            if A == 0:
                yield from samples(g, t)
            yield pub(("GATE", g, k), tag + 1)

    agents = [head(g, j, p) for g in range(G) for j in range(NH) for p in range(2)]
    agents += [unit(g, k) for g in range(G) for k in range(NU)]
    speed = [rng.random() ** 4 + 0.002 for _ in agents]     # some agents hundreds of times slower
    cur = [next(a) for a in agents]
    live = set(range(len(agents)))
    waiting = {}                                            # word -> agents whose wait on it failed
    ready = set(live)

    def holds(i):
        kind, key, tag = cur[i]
        if kind in ("w", "arrive"):
            return True
        x = mem.get(key, 0)
        if kind == "sync":
            return x >= tag
        return (x & 1) == (tag & 1) if kind == "r1" else (x & 0xFFFF) == (tag & 0xFFFF)

    for _ in range(max_ticks):
        if not live:
            return None
        if not ready:
            stuck = [(cur[i], mem.get(cur[i][1], 0)) for i in sorted(live)][:4]
            return f"deadlock (a word lost or never written): {stuck}"
        rd = list(ready)
        i = rng.choices(rd, weights=[speed[x] for x in rd])[0]
        kind, key, tag = cur[i]
        if not holds(i):
            ready.discard(i)
            waiting.setdefault(key, set()).add(i)
            continue
        if kind in ("w", "arrive"):
            mem[key] = tag if kind == "w" else mem.get(key, 0) + 1
            ready |= waiting.pop(key, set())
        elif kind != "sync" and mem.get(key, 0) != tag:
            return f"misread: {key} awaited at step tag {tag}, holds {mem.get(key, 0)}"
        try:
            cur[i] = next(agents[i])
        except StopIteration:
            live.discard(i)
            ready.discard(i)
    return "ran out of ticks"


MODES = [("ALL", 8, 2), ("ALL", 4, 4), ("SLICE", 2, 8)]


@pytest.mark.parametrize("mode,G,L", MODES)
@pytest.mark.parametrize("A", [0, 1, 2, 3])
def test_exchange_protocol_has_no_lost_or_misread_word(mode, G, L, A):
    """Random interleavings, skewed speeds: every awaited word is read with
    the step it was awaited for, and nothing waits forever (B = 16 lanes of
    one utterance over the groups, horizon 4, the kernel's slot count)."""
    fails = [(sd, e) for sd in range(6) for e in [run(mode, G=G, L=L, A=A, seed=sd)] if e]
    assert not fails, fails[:2]


@pytest.mark.parametrize("mode", ["ALL", "SLICE"])
def test_groups_without_sample_words(mode):
    """Utterances (no words between groups): one group, many steps."""
    G, L = 1, (8 if mode == "SLICE" else 2)
    fails = [(sd, e) for sd in range(30) for e in [run(mode, G=G, L=L, B=1, F=0, A=0, rows=60, seed=sd)] if e]
    assert not fails, fails[:2]


@pytest.mark.parametrize("mode,G,L", MODES)
def test_the_model_catches_a_wave_that_publishes_on_its_own_words(mode, G, L):
    """A wave that replaces y_c once its own words are there (and not every
    unit's) loses a word for a unit that has not read the old y_c."""
    assert any((run(mode, G=G, L=L, A=1, guard=False, seed=sd) or "").startswith("deadlock") for sd in range(12))
    assert any((run(mode, G=1, L=L, B=1, F=0, A=0, rows=60, guard=False, seed=sd) or "").startswith("deadlock")
               for sd in range(40))


def test_the_model_catches_a_reused_sample_slot():
    """The model is not blind: with too few sample slots (SS = 2 at A = 1) or
    without idle lanes publishing, some interleaving loses a sample word."""
    assert any(run("ALL", A=1, SS=2, seed=sd) for sd in range(40))
    assert any(run("ALL", A=1, idle_publish=False, seed=sd) for sd in range(40))
