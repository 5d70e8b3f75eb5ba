"""Leaf records of the two-lanes-per-child kernel (values and errors staged
through LDS, the product integrals of the box basis or the pairs of a general
set) against the one-wave-per-parent kernel, which stores pairs itself: the
same rule sums in another rounding order.  Tolerances: a rectangle's pair is a
sum of 81 products, each side's rounding below 81 x 2^-53 = 9e-15 of the sum
of their magnitudes, which is at most ~10 times the largest pair here: 1e-12
of it is the rectangle bar of the oracle tests; integrals of the same
containers agree within the tolerance they are integrated to."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

ROW, Q = [1.0, -0.3, -1.1, 0.05, 0.3], [2.88, 0.26]


def sets():
    r = np.random.default_rng(11)
    full = np.linalg.qr(r.normal(size=(9, 9)))[0]
    return {"box": (W.ff_box(1), 1), "five": (W.ff5(), 1), "one": (W.ff_box(0), 0),
            "minus one": (-W.ff_box(0), 0), "general 6": (full[:6].copy(), 1),
            "general 7": (full[:7].copy(), 1), "general 9": (full.copy(), 1)}


@pytest.fixture(scope="module")
def P():
    import paid_1610_09991_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("name", list(sets()))
@pytest.mark.parametrize("n", [1, 7, 8, 9, 65])
def test_rectangles_of_both_kernels(P, name, n):
    """n parents: part of a wave's eight, exactly eight, a remainder, many waves"""
    ff, L = sets()[name]
    rng = np.random.default_rng(n)
    d = rng.integers(0, 9, n)
    codes = np.stack([d, rng.integers(0, 2 ** d), rng.integers(0, 2 ** d)], axis=1)
    for ch in (P.PP, P.PH):
        got = []
        for layout in (0, 1):
            with P.Context(eval_layout=layout) as c:
                got.append(c.children(ROW, Q, ch, ff, L, codes))
        (q0, k0), (q1, k1) = got
        big = np.abs(q1).max(axis=-1, keepdims=True)
        assert (np.abs(q0 - q1) <= 1e-12 * big).all()
        assert (np.abs(k0 - k1) <= 1e-12 * np.abs(q1).sum(axis=-1) + 1e-7 * k1).all()


@pytest.mark.parametrize("name", list(sets()))
@pytest.mark.parametrize("mode", ["global", "per_integral", "weighted"])
def test_errors_and_values_of_both_kernels(P, name, mode):
    """stored per-pair errors (err=True) in every error mode"""
    ff, L = sets()[name]
    M = len(ff)
    em = {"global": P.ERR_GLOBAL, "per_integral": P.ERR_PER_INTEGRAL, "weighted": P.ERR_WEIGHTED}[mode]
    q = np.array([Q, [0.0, 0.0], [1.57, 1.31]])
    w = np.random.default_rng(2).uniform(0.1, 1.0, (6, M, M))
    got = []
    for layout in (0, 1):
        with P.Context(eval_layout=layout, err_mode=em, max_regions=1 << 16) as c:
            if mode == "weighted":
                c.set_pair_weights(w)
            got.append(c.integrate([ROW], q, ff, L, rtol=1e-6, err=True))
    (a, ea, sa, ra), (b, eb, sb, rb) = got
    assert ra == P.OK and rb == P.OK
    big = np.abs(b).max(axis=(-1, -2), keepdims=True)
    assert (np.abs(a - b) <= 1e-6 * big).all()
    # the error sums of trees of the same size (a split decided by the last
    # bits of a key moves single leaves between them)
    assert abs(sa["regions"] - sb["regions"]) <= 0.01 * sb["regions"] + 8
    assert (np.abs(ea - eb) <= 0.05 * eb + 1e-9 * big).all()
