"""The evaluation's share-out of a round's work items: every workgroup takes
a first chunk by its index and then chunks from a counter.  Checked on the
host (the same arithmetic as the kernel, in Python): whatever the order in
which workgroups come back to the counter, every item is taken exactly once
and every workgroup ends; and on the GPU, results do not depend on the number
of workgroups."""
import random

import numpy as np
import pytest

import workloads as W


def chunk_items(left, unit, waves, grid):
    wg = unit * waves
    half = left // (2 * grid)
    if half >= wg:
        return half // wg * wg
    even = (left + grid - 1) // grid
    return max(unit, min(wg, (even + unit - 1) // unit * unit))


@pytest.mark.parametrize("unit,waves", [(1, 4), (1, 1), (8, 4), (8, 8)])
@pytest.mark.parametrize("total", [0, 1, 7, 8, 9, 300, 8191, 24577, 1000003])
def test_every_item_is_taken_once(unit, waves, total):
    rng = random.Random(total + unit)
    for grid in (1, 3, 256, 768):
        taken, counter = [], 0
        c0 = chunk_items(total, unit, waves, grid)
        alive = []
        for b in range(grid):
            i0 = min(b * c0, total)
            if i0 < min(i0 + c0, total):
                taken.append((i0, min(i0 + c0, total)))
                alive.append(b)
        base = c0 * grid
        while alive:
            k = rng.randrange(len(alive))
            # the counter may have moved between its reading and the addition
            seen = base + max(0, counter - rng.choice([0, 0, unit * waves]))
            if base >= total or seen >= total:
                alive.pop(k)
                continue
            c = chunk_items(total - seen, unit, waves, grid)
            i0, counter = base + counter, counter + c
            if i0 >= total:
                alive.pop(k)
                continue
            taken.append((i0, min(i0 + c, total)))
        taken.sort()
        assert sum(b - a for a, b in taken) == total
        assert all(taken[i][1] == taken[i + 1][0] for i in range(len(taken) - 1))


@pytest.mark.gpu
@pytest.mark.parametrize("layout", [0, 1])
def test_results_do_not_depend_on_the_number_of_workgroups(layout):
    """rounds of one item up to thousands, two parameter rows (two tables a
    call), on one workgroup per compute unit and on as many as fit"""
    import paid_1610_09991_amd as P
    p = [[1.0, -0.25, -0.95, 0.05, 0.3], [1.0, -0.1, -0.4, 0.08, 1.0]]
    q = W.q_grid(16)[::41]
    ref = None
    for wg in (0, 1, 7):
        with P.Context(max_regions=1 << 14, eval_layout=layout, eval_wg_per_cu=wg) as c:
            out, _, st, rc = c.integrate(p, q, W.ff_box(1), 1, rtol=1e-6)
        assert rc == P.OK
        if ref is None:
            ref = out, st["regions"]
        assert np.array_equal(out, ref[0]) and st["regions"] == ref[1]


@pytest.mark.gpu
@pytest.mark.parametrize("err_mode,err", [(0, False), (0, True), (1, False)])
@pytest.mark.parametrize("basis", ["box0", "box1", "five", "mixed"])
def test_groups_of_one_item_hold_the_same_values(basis, err_mode, err):
    """a round of at most as many items as waves is taken in groups of one item,
    otherwise of eight: the same sums in the same order.  With seven times the
    workgroups some round (each has about four times the items of the one
    before) is of the one kind here and of the other there."""
    import paid_1610_09991_amd as P
    if basis == "mixed":
        ff, L = np.linalg.qr(np.random.default_rng(5).normal(size=(9, 9)))[0][:4].copy(), 1
    else:
        ff, L = (W.ff5(), 1) if basis == "five" else (W.ff_box(int(basis[-1])), int(basis[-1]))
    p = [[1.0, -0.25, -0.95, 0.03, 0.1]]
    for q in (W.q_grid(16)[37:38], W.q_grid(16)[::29]):
        got = []
        for wg in (1, 7):
            with P.Context(max_regions=1 << 18, pool_gib=16, eval_wg_per_cu=wg, err_mode=err_mode) as c:
                out, e, st, rc = c.integrate(p, q, ff, L, rtol=1e-6, err=err)
            assert rc == P.OK
            got.append((out, e, st["regions"]))
        assert np.array_equal(got[0][0], got[1][0]) and got[0][2] == got[1][2]
        assert not err or np.array_equal(got[0][1], got[1][1])


# ------------------------------------------------------------------ slots of items
def wave_slot(woff, W, g):
    lo, hi = 0, W
    while hi - lo > 1:
        step = (hi - lo + 63) >> 6
        c = sum(1 for lane in range(64) if lo + (lane + 1) * step < hi and woff[lo + (lane + 1) * step] <= g)
        lo += c * step
        hi = min(lo + step, hi)
    return lo


def group_items(woff, W, g0, gend):
    """slot and place of each of the eight lane groups' items, as the wave forms them"""
    s = wave_slot(woff, W, g0)
    off = [woff[min(s + 1 + lane, W)] for lane in range(64)]
    out = []
    for it in range(8):
        w = min(g0 + it, gend - 1)
        mine = sum(1 for o in off if o <= w)
        prev = off[max(mine - 1, 0)]
        lo, t = (prev if mine else woff[s]), s + mine
        while mine == 64 and woff[t + 1] <= w:
            t += 1
            lo = woff[t]
        out.append((t, w - lo))
    return out


@pytest.mark.parametrize("W", [1, 2, 3, 63, 64, 65, 66, 700, 4097, 5000])
@pytest.mark.parametrize("fill", [0.02, 0.5, 1.0])
def test_slots_of_items(W, fill):
    """against the definition (slot t holds items woff[t]..woff[t + 1] - 1), with
    runs of empty slots longer than the 64 offsets a wave reads at a time"""
    rng = np.random.default_rng(W)
    cnt = np.where(rng.random(W) < fill, rng.integers(1, 40, W), 0)
    cnt[rng.integers(0, W)] += 5
    woff = np.concatenate([[0], np.cumsum(cnt)]).tolist()
    total = woff[-1]
    slot = np.repeat(np.arange(W), cnt)
    for g0 in list(range(0, min(total, 200))) + rng.integers(0, total, 100).tolist():
        assert wave_slot(woff, W, g0) == slot[g0]
        gend = min(total, g0 + int(rng.integers(1, 20)))
        for it, (t, r) in enumerate(group_items(woff, W, g0, gend)):
            w = min(g0 + it, gend - 1)
            assert t == slot[w] and r == w - woff[t] and 0 <= r < cnt[t]


def row_end(woff, entry, W, s, i1):
    for t0 in range(s + 1, W, 64):
        past = False
        for t in range(t0, t0 + 64):
            lo, up = (woff[t], woff[t + 1]) if t < W else (i1, i1)
            if lo < i1 and up > lo and entry[t] != entry[s]:
                return lo
            past |= lo >= i1
        if past:
            break
    return i1


@pytest.mark.parametrize("W", [1, 5, 64, 65, 129, 1000])
def test_runs_of_one_parameter_row(W):
    rng = np.random.default_rng(W + 1)
    cnt = np.where(rng.random(W) < 0.4, rng.integers(1, 9, W), 0)
    cnt[0] += 1
    woff = np.concatenate([[0], np.cumsum(cnt)]).tolist()
    entry = np.sort(rng.integers(0, 1 + W // 20, W))
    row = np.repeat(entry, cnt)
    slot = np.repeat(np.arange(W), cnt)
    for g in rng.integers(0, woff[-1], 200):
        i1 = int(min(woff[-1], g + rng.integers(1, 500)))
        want = g
        while want < i1 and row[want] == row[g]:
            want += 1
        assert row_end(woff, entry, W, int(slot[g]), i1) == want
