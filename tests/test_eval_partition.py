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
