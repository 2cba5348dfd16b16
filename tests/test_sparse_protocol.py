"""A CPU model of the block-sparse kernel's exchange protocol (CPU only; the
kernel is in wr_persist.hip: heads with split output MLPs and sparse units).

NK coarse heads hold the coarse gates and the coarse MLP, NK fine heads the fine
ones; every head draws both bytes.  A unit's rows lie in one half, so its
gate words are read by the heads of that half alone.  Agents run the kernel's
order of publishes and waits, one read of one word per scheduling step, under
random interleavings with strongly skewed speeds.  Words carry the kernel's tags:

* single-buffered words (y_f slices, gate words) hold the parity of step + 1;
* double-buffered words (y_c slices, coarse and fine partial logits) of step s
  sit in buffer s mod 2 and hold the parity of s / 2 + 1.

Two buffers, because nothing else keeps a coarse head from running one step
ahead of another head's read of its partial logits (the fine heads' words that
let it go on follow its own partials, not that head's read), of a fine row's unit's
read of its y_c (whose words the fine heads wait for, a step later), and a
fine head ahead of another fine head in the same way.  A coarse head at step s + 2
has waited for every coarse-row unit's words, which follow every fine head's
y_f of step s + 1, which follow every fine-row unit's words of step s + 1 and
every coarse head's partials of step s + 1: all that read a word of step s is done.

A reader accepts a word whose bit matches, and the model then checks that the
word was written for the awaited step: a match on another step is a misread; a
word replaced before it was read is a deadlock.

What the model leaves out: values, barriers inside a workgroup, memory
ordering of the hardware (every write is visible to the next read) and the
bounded waits' clock.
"""
import random

import pytest


def run(NK=2, NU=3, T=30, seed=0, wide=True, yc=True, pc=True, pf=True, max_ticks=400_000):
    """NK heads and NU units a half; wide: the fine gate words are read before the step (GU > 1), else
    after c_t; yc, pc, pf: double-buffered."""
    rng = random.Random(seed)
    mem = {}

    def word(name, i, s):
        if {"YC": yc, "PC": pc, "PF": pf}.get(name, False):
            return (name, i, s & 1), ((s >> 1) + 1) & 1
        return (name, i), (s + 1) & 1

    def pub(name, i, s):
        return ("w", *word(name, i, s), s)

    def wait(name, n, s):
        for i in range(n):
            yield ("r", *word(name, i, s), s)

    def coarse_head(j):
        yield from wait("GA", NU, 0)
        for s in range(T):
            yield pub("YC", j, s)
            yield pub("PC", j, s)
            yield from wait("PC", NK, s)
            yield from wait("PF", NK, s)
            if s + 1 < T:
                yield from wait("GA", NU, s + 1)

    def fine_head(j):
        if wide:
            yield from wait("GF", NU, 0)
        for s in range(T):
            yield from wait("PC", NK, s)
            if not wide:
                yield from wait("GF", NU, s)
            yield pub("YF", j, s)
            yield pub("PF", j, s)
            yield from wait("PF", NK, s)
            if wide and s + 1 < T:
                yield from wait("GF", NU, s + 1)

    def unit(name, k):
        yield pub(name, k, 0)
        for t in range(T - 1):
            yield from wait("YC", NK, t)
            yield from wait("YF", NK, t)
            yield pub(name, k, t + 1)

    agents = [coarse_head(j) for j in range(NK)] + [fine_head(j) for j in range(NK)]
    agents += [unit(n, k) for n in ("GA", "GF") for k in range(NU)]
    speed = [rng.random() ** 4 + 0.002 for _ in agents]     # some agents hundreds of times slower
    cur = [next(a) for a in agents]
    live = set(range(len(agents)))
    for _ in range(max_ticks):
        if not live:
            return None
        rd = [i for i in live if cur[i][0] == "w" or mem.get(cur[i][1], (0, -1))[0] == cur[i][2]]
        if not rd:
            return f"deadlock (a word lost or never written): {[cur[i] for i in sorted(live)][:4]}"
        i = rng.choices(rd, weights=[speed[x] for x in rd])[0]
        kind, key, bit, s = cur[i]
        if kind == "w":
            mem[key] = (bit, s)
        elif mem[key][1] != s:
            return f"misread: {key} awaited for step {s}, holds step {mem[key][1]}"
        try:
            cur[i] = next(agents[i])
        except StopIteration:
            live.discard(i)
    return "ran out of ticks"


@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("NK,NU", [(2, 3), (3, 2), (1, 2), (4, 4)])
def test_sparse_protocol_has_no_lost_or_misread_word(wide, NK, NU):
    """Random interleavings, skewed speeds: every awaited word is read with the
    step it was awaited for, and nothing waits forever."""
    fails = [(sd, e) for sd in range(40) for e in [run(NK=NK, NU=NU, wide=wide, seed=sd)] if e]
    assert not fails, fails[:2]


@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("one", ["yc", "pc", "pf"])
def test_the_model_catches_single_buffered_words(wide, one):
    """With y_c or either half's partial logits in one buffer some interleaving loses a word."""
    assert any(run(wide=wide, seed=sd, **{one: False}) for sd in range(60))
