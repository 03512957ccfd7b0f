"""The exchange of the resident tridiagonalisation (csrc/trd.hip) on the host.

A model of its protocol: per column c every work-group publishes its part of
y = A v and, if it owns column c + 1, that column, then gathers both.  Nothing
orders a work-group that owns no column above c any more, so any work-group may
be held back by any amount.  Every gathered value has to be the one of its
column.  The slots are those of csrc/trd_slot.h, compiled here."""
import ctypes
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = """
#include "{header}"
extern "C" size_t slot(int n, int c) {{ return zk::trd_slot(n, c); }}
extern "C" size_t next(int n) {{ return zk::trd_slot_next(n); }}
extern "C" size_t doubles(int n) {{ return zk::trd_slot_doubles(n); }}
"""


@pytest.fixture(scope="module")
def slots(tmp_path_factory):
    d = tmp_path_factory.mktemp("slot")
    src, lib = d / "s.cpp", d / "s.so"
    src.write_text(SRC.format(header=os.path.join(os.path.dirname(HERE), "paper_2402_11868_amd", "csrc", "trd_slot.h")))
    subprocess.check_call(["g++", "-O1", "-fPIC", "-shared", str(src), "-o", str(lib)])
    so = ctypes.CDLL(str(lib))
    for f in (so.slot, so.next, so.doubles):
        f.restype = ctypes.c_size_t
    return so


def _run(n, per, slot, nxt, recycle, order):
    """All work-groups to their end; `order` picks which runnable one goes on.
    Returns the gathered values that were not their column's, and the
    work-groups left waiting."""
    G = -(-n // per)
    mem, wrong = {}, []

    def group(g):
        mine = range(g, n, G)
        for c in range(n - 1):
            y, a = slot(c), slot(c) + nxt
            if (c + 1) % G == g:
                mem.update((a + 2 * i, ("a", c, i)) for i in range(c + 1, n))
            mem.update((y + 2 * j, ("y", c, j)) for j in mine if j > c)
            yield
            for i in range(c + 1, n):
                for at, kind in ((y + 2 * i, "y"), (a + 2 * i, "a")):
                    while at not in mem:
                        yield "wait"
                    if mem[at] != (kind, c, i):
                        wrong.append((g, kind, c, i, mem[at]))
            if recycle and c > 0:   # the owners empty what everybody is thought to have read
                y, a = slot(c - 1), slot(c - 1) + nxt
                for j in mine:
                    if j >= c:
                        mem.pop(y + 2 * j, None)
                if c % G == g:
                    for i in range(c, n):
                        mem.pop(a + 2 * i, None)
            yield

    live = {g: group(g) for g in range(G)}
    waiting = {}
    while live:
        g = order([h for h in live if waiting.get(h) != len(mem)] or list(live))
        got = next(live[g], "end")
        if got == "end":
            del live[g]
        waiting[g] = len(mem) if got == "wait" else None
        if live and all(waiting.get(h) == len(mem) for h in live):
            break   # nobody can go on
    return wrong, sorted(live)


def _held_back(victim):
    return lambda can: next((g for g in can if g != victim), victim)


@pytest.mark.parametrize("n,per", [(9, 8), (17, 8), (24, 4), (33, 4)])
def test_any_work_group_may_be_held_back(slots, n, per):
    def slot(c):
        return slots.slot(n, c)
    G = -(-n // per)
    for victim in range(G):
        assert _run(n, per, slot, slots.next(n), False, _held_back(victim)) == ([], [])
    rng = random.Random(n)
    for _ in range(5):
        assert _run(n, per, slot, slots.next(n), False, rng.choice) == ([], [])


def test_the_model_sees_a_recycled_slot(slots):
    """Three slots used in turn and emptied by their owners: a work-group that
    owns none of the last columns and is held back reads another column's
    values or waits for ever."""
    n, per = 24, 4
    bad = [_run(n, per, lambda c: 4 * n * (c % 3), slots.next(n), True, _held_back(v)) for v in range(6)]
    assert any(w or left for w, left in bad)


@pytest.mark.parametrize("n", [129, 256, 257, 1024, 2048])
def test_slots_are_disjoint_and_fit(slots, n):
    at = [slots.slot(n, c) for c in range(n - 1)]
    size = slots.next(n) + 2 * n
    assert slots.next(n) >= 2 * n
    assert all(b - a >= size for a, b in zip(at, at[1:]))
    assert at[-1] + size <= slots.doubles(n) <= 5 * n * n   # the inverse-iteration scratch
