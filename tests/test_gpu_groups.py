"""Rectangles of the two-lanes-per-child kernel in both of its shapes: groups of
eight parents (a call of several), with idle lanes and several waves where the
number is no multiple of eight, and groups of one (a call of one).  The same sums
in the same order: equal bits; and the groups of eight against the oracle, to
1e-12 of a rectangle's largest pair as in its other rectangle tests."""
import math

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

ROW, Q = (1.0, -0.3, -1.1, 0.05, 0.3), (2.88, 0.26)


@pytest.fixture(scope="module")
def P():
    import paid_1610_09991_amd as P
    P.lib()
    return P


def sets():
    full = np.linalg.qr(np.random.default_rng(11).normal(size=(9, 9)))[0]
    return {"box": (W.ff_box(1), 1), "five": (W.ff5(), 1), "one": (W.ff_box(0), 0),
            "general 6": (full[:6].copy(), 1)}


def parents(n):
    rng = np.random.default_rng(n)
    d = rng.integers(0, 9, n)
    return np.stack([d, rng.integers(0, 2 ** d), rng.integers(0, 2 ** d)], axis=1)


@pytest.mark.parametrize("name", list(sets()))
@pytest.mark.parametrize("n", [2, 7, 8, 9, 63, 64, 65, 130, 600])
def test_groups_of_eight_and_of_one_agree(P, name, n):
    ff, L = sets()[name]
    codes = parents(n)
    with P.Context() as c:
        for ch in (P.PP, P.PH):
            q8, k8 = c.children(ROW, Q, ch, ff, L, codes)
            for i in range(0, n, 1 if n < 100 else 13):
                q1, k1 = c.children(ROW, Q, ch, ff, L, codes[i:i + 1])
                assert np.array_equal(q1[0], q8[i]) and np.array_equal(k1[0], k8[i]), i


@pytest.mark.parametrize("name", list(sets()))
@pytest.mark.parametrize("n", [1, 13, 70])
def test_groups_match_oracle_rectangles(P, name, n):
    ff, L = sets()[name]
    codes = parents(n)
    for ch, och in ((P.PP, O.PP), (P.PH, O.PH)):
        with P.Context() as c:
            q2n, keys = c.children(ROW, Q, ch, ff, L, codes)
        oc = O.Container(ff, L, t=ROW[0], tp=ROW[1], mu=ROW[2], T=ROW[3], Omega=ROW[4], lx=Q[0], ly=Q[1],
                         channel=och)
        for i, (d, ix, iy) in enumerate(codes):
            w = 2 * math.pi / 2 ** d
            for k in range(4):
                x0, y0 = -math.pi + ix * w + (k & 1) * w / 2, -math.pi + iy * w + (k >> 1) * w / 2
                qn, ref = oc.region(x0, x0 + w / 2, y0, y0 + w / 2)
                assert np.abs(q2n[i, k] - ref).max() <= 1e-12 * np.abs(ref).max(), (i, k)
                e = np.abs(qn - ref).sum()
                assert abs(keys[i, k] - e) <= 1e-12 * np.abs(ref).sum() + 1e-7 * e, (i, k)
