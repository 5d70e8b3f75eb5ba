"""The evaluation's share-out of a round's work items, from the functions that
the kernels call (csrc/share.h, built here for the host).  Whatever the order in
which workgroups and waves come to the counters, every item is taken exactly once,
every group lies in one parameter row, and every wave ends.  The waves run as
coroutines that give way at each atomic operation, in random order; the protocol
around the arithmetic (range, lock, mode, the change of the table at a barrier)
is written out as in k_children_lpc and k_children."""
import ctypes as C
import os
import random
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
XCDS = 8

WRAP = r"""
#define __host__
#define __device__
#include "share.h"
using namespace paid;
extern "C" {
void span_first_chunk(int t, int w, int g, int b, int *o) { Span k = first_chunk(t, w, g, b); o[0] = k.i0; o[1] = k.i1; }
long base_chunk(int t, int w, int g) { return chunk_base(t, w, g); }
int items_chunk(int l, int w, int g) { return chunk_items(l, w, g); }
void xcd(int t, int g, int b, int n, int *o) {
  XcdShare s = xcd_share(t, g, b, n);
  o[0] = s.x; o[1] = s.first; o[2] = s.last; o[3] = s.wgs; o[4] = s.index;
}
int items_share(int l, int gr, int g, int n) { return share_items(l, gr, g, n); }
void span_first_share(const int *x, int c, int *o) {
  XcdShare s{x[0], x[1], x[2], x[3], x[4]};
  Span k = first_share(s, c); o[0] = k.i0; o[1] = k.i1; o[2] = share_base(s, c);
}
void span_counted(int b, int t, int n, int c, int *o) { Span k = counted_span(b, t, n, c); o[0] = k.i0; o[1] = k.i1; }
unsigned long long word(int a, int b) { return range_word(Span{a, b}); }
int empty(unsigned long long r) { return range_empty(r); }
void group(unsigned long long r, int n, int *o) { Span k = range_group(r, n); o[0] = k.i0; o[1] = k.i1; }
}
"""


@pytest.fixture(scope="module")
def S(tmp_path_factory):
    d = tmp_path_factory.mktemp("share")
    src, so = d / "share.cpp", d / "share.so"
    src.write_text(WRAP)
    inc = os.path.join(ROOT, "paid_1610_09991_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-fPIC", "-shared", "-I", inc, str(src), "-o", str(so)],
                   check=True)
    L = C.CDLL(str(so))
    L.base_chunk.restype = C.c_long
    L.word.restype = C.c_ulonglong
    L.empty.argtypes = [C.c_ulonglong]
    L.group.argtypes = [C.c_ulonglong, C.c_int, C.c_void_p]
    return L


def ints(f, n, *a):
    o = (C.c_int * n)()
    f(*a, o)
    return list(o)


def covered(taken, total):
    taken = sorted(taken)
    assert sum(b - a for a, b in taken) == total
    assert all(x[1] == y[0] for x, y in zip(taken, taken[1:]))


@pytest.mark.parametrize("waves", [1, 4, 7])
@pytest.mark.parametrize("total", [0, 1, 9, 300, 8191, 24577, 1000003])
def test_chunks_of_one_counter(S, waves, total):
    rng = random.Random(total + waves)
    for grid in (1, 3, 256, 769):
        taken, counter = [], 0
        alive = []
        for b in range(grid):
            k = ints(S.span_first_chunk, 2, total, waves, grid, b)
            if k[0] < k[1]:
                taken.append(tuple(k))
                alive.append(b)
        base = S.base_chunk(total, waves, grid)
        while alive:
            i = rng.randrange(len(alive))
            # the counter may have moved between its reading and the addition
            seen = base + max(0, counter - rng.choice([0, 0, waves]))
            if base >= total or seen >= total:
                alive.pop(i)
                continue
            c = S.items_chunk(total - seen, waves, grid)
            k = ints(S.span_counted, 2, base, total, counter, c)
            counter += c
            if k[0] >= k[1]:
                alive.pop(i)
                continue
            taken.append(tuple(k))
        covered(taken, total)


class Workgroup:
    """One workgroup of k_children_lpc: its waves are generators that yield
    before every shared access ("go") and at the barriers ("barrier")."""

    def __init__(self, S, total, rows, grid, block, waves, group, counters, taken):
        self.S, self.rows, self.grid, self.group = S, rows, grid, group
        self.counters, self.taken, self.waves = counters, taken, waves
        x = ints(S.xcd, 5, total, grid, block, XCDS)
        c = S.items_share(x[2] - x[1], group, grid, XCDS)
        self.xcd = x[0]
        self.rest, self.end, self.base = ints(S.span_first_share, 3, (C.c_int * 5)(*x), c)
        self.total = x[2]
        self.idle = self.rest >= self.end
        self.range, self.lock, self.mode, self.row, self.next = 0, 0, 0, -1, (0, 0)

    def next_range(self, loaded):
        k = [self.rest, self.end]
        if k[0] >= k[1]:
            if self.base < self.total:
                yield "go"
                seen = self.base + self.counters[self.xcd]
                if seen < self.total:
                    c = self.S.items_share(self.total - seen, self.group, self.grid, XCDS)
                    yield "go"
                    k = ints(self.S.span_counted, 2, self.base, self.total, self.counters[self.xcd], c)
                    self.counters[self.xcd] += c
        if k[0] >= k[1]:
            self.mode = 2
            return
        e = self.rows[k[0]]
        hi = k[0]
        while hi < k[1] and self.rows[hi] == e:
            hi += 1
        self.rest, self.end = hi, k[1]
        if e == loaded:
            yield "go"
            self.range = self.S.word(k[0], hi)
        else:
            self.row, self.next = e, (k[0], hi)
            yield "go"
            self.mode = 1

    def take_group(self, loaded):
        while True:
            yield "go"
            r = self.range
            if not self.S.empty(r):
                yield "go"
                r = self.range
                self.range += self.group
            yield "go"
            mode = self.mode
            if not self.S.empty(r):
                return ints(self.S.group, 2, r, self.group)
            if mode:
                return None
            yield "go"
            if self.lock == 0:
                self.lock = 1
                yield "go"
                if self.S.empty(self.range) and self.mode == 0:
                    yield from self.next_range(loaded)
                yield "go"
                self.lock = 0

    def wave(self, w):
        if w == 0:
            yield from self.next_range(-1)
        while True:
            yield "barrier"
            if self.mode == 2:
                return
            e = self.row
            yield "barrier"
            if w == 0:
                self.range = self.S.word(*self.next)
                self.mode = 0
            yield "barrier"
            while True:
                k = yield from self.take_group(e)
                if k is None:
                    break
                assert 0 < k[1] - k[0] <= self.group and all(self.rows[i] == e for i in range(*k))
                self.taken.append(tuple(k))


def run(wgs, rng):
    """all workgroups at once, a random wave one step at a time; a wave at a
    barrier waits for the others of its workgroup"""
    live = {}
    for b, g in enumerate(wgs):
        for w in range(g.waves):
            live[b, w] = g.wave(w)
    at, left = {b: set() for b in range(len(wgs))}, {b: g.waves for b, g in enumerate(wgs)}
    ready, steps = list(live), 0
    while ready:
        steps += 1
        assert steps < 2_000_000, "a wave never ends"
        i = rng.randrange(len(ready))
        ready[i], ready[-1] = ready[-1], ready[i]
        b, w = ready.pop()
        try:
            what = next(live[b, w])
        except StopIteration:
            left[b] -= 1
            what = None
        if what == "go":
            ready.append((b, w))
            continue
        if what == "barrier":
            at[b].add(w)
        if at[b] and len(at[b]) == left[b]:
            ready += [(b, v) for v in at[b]]
            at[b] = set()
    assert not any(at.values()) and not any(left.values())


@pytest.mark.parametrize("grid", [1, 2, 7, 8, 9, 30])
@pytest.mark.parametrize("total", [0, 1, 5, 8, 31, 64, 700, 3001])
@pytest.mark.parametrize("group", [1, 8])
def test_shares_of_the_xcds(S, grid, total, group):
    """grids below eight and no multiple of it, fewer items than workgroups,
    runs of one parameter row shorter and longer than a share"""
    for waves, n_rows, seed in ((1, 1, 0), (3, 4, 1), (8, 1, 2), (4, 40, 3)):
        rng = random.Random(1000 * grid + total + seed)
        cuts = sorted(rng.randrange(total + 1) for _ in range(n_rows - 1))
        rows = np.searchsorted(cuts, np.arange(total), side="right").tolist()
        counters, taken = [0] * XCDS, []
        wgs = [Workgroup(S, total, rows, grid, b, waves, group, counters, taken) for b in range(grid)]
        run([g for g in wgs if not g.idle], rng)
        covered(taken, total)


@pytest.mark.parametrize("total", [2 ** 31 - 1, 2 ** 31 - 9, 1_500_000_001])
@pytest.mark.parametrize("grid", [1, 768, 2048])
def test_the_largest_rounds(S, total, grid):
    """no intermediate value overflows (undefined behaviour ends the test program),
    and the first shares and the counters' parts tile the round"""
    for group in (1, 8):
        taken = []
        for b in range(grid):
            x = ints(S.xcd, 5, total, grid, b, XCDS)
            c = S.items_share(x[2] - x[1], group, grid, XCDS)
            lo, hi, base = ints(S.span_first_share, 3, (C.c_int * 5)(*x), c)
            if lo < hi:
                taken.append((lo, hi))
            if x[4] == 0 and base < x[2]:
                taken.append((base, x[2]))
        covered(taken, total)
    assert ints(S.group, 2, S.word(total - 3, total), 8) == [total - 3, total]
