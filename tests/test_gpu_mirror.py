"""Mirror images together (both bubbles are even under p -> -p, so a leaf with
p_y >= 0 stands for itself and its image) against the full tree, which the
library grows when its leaves are asked for one by one.  The two select the
same leaves up to which of equal keys come first, so the trees have the same
size to a few splits; both meet the tolerance rtol in the sum over pairs, so
values differ by at most 2 rtol of that sum, and pairs of odd joint parity, rounding noise on the full tree,
are exact zeros."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

ROWS = [[1.0, -0.25, -0.95, 0.05, 0.3], [1.0, -0.1, -0.4, 0.08, 1.0]]
Q = np.array([[2.88, 0.26], [0.0, 0.0], [1.57, 1.31], [7.5, -13.0], [np.pi, -np.pi]])


@pytest.fixture(scope="module")
def P():
    import paid_1610_09991_amd as P
    P.lib()
    return P


def sets():
    full = np.linalg.qr(np.random.default_rng(11).normal(size=(9, 9)))[0]
    return {"box1": (W.ff_box(1), 1), "five": (W.ff5(), 1), "general": (full[:6].copy(), 1),
            "one": (W.ff_box(0), 0), "box2": (W.ff_box(2), 2)}


def both(P, ff, L, rtol, model=None, err=False, weights=None, **kw):
    """(mirror images together, full tree): out, err, stats, code"""
    n = len(ROWS) * len(Q) * 2
    MU = len(ff) * (len(ff) + 1) // 2
    got = []
    for full in (False, True):
        with P.Context(max_regions=1 << 16, **kw) as c:
            if model is not None:
                c.set_seed_model(model, kappa=1.0)
            if weights is not None:
                c.set_pair_weights(weights)
            if full:
                c.set_leaf_output(np.zeros((n, 1, 3), dtype=np.int32), np.zeros((n, 1, MU)))
            got.append(c.integrate(ROWS, Q, ff, L, rtol=rtol, err=err))
    return got


@pytest.mark.parametrize("name", list(sets()))
@pytest.mark.parametrize("mode", ["global", "per_integral", "weighted"])
def test_images_together_match_the_full_tree(P, name, mode):
    ff, L = sets()[name]
    M, rtol = len(ff), 1e-6
    em = {"global": P.ERR_GLOBAL, "per_integral": P.ERR_PER_INTEGRAL, "weighted": P.ERR_WEIGHTED}[mode]
    w = np.random.default_rng(2).uniform(0.1, 1.0, (20, M, M)) if mode == "weighted" else None
    (a, ea, sa, ra), (b, eb, sb, rb) = both(P, ff, L, rtol, err_mode=em, err=True, weights=w)
    assert ra == P.OK and rb == P.OK
    l1 = np.abs(b).sum(axis=(-1, -2), keepdims=True)
    assert (np.abs(a - b) <= 2 * rtol * l1).all()
    assert abs(sa["regions"] - sb["regions"]) <= 0.02 * sb["regions"]
    assert abs(sa["kernel_evals"] - sb["kernel_evals"]) <= 0.02 * sb["kernel_evals"]
    assert sa["max_depth"] == sb["max_depth"] or mode == "weighted"
    assert np.array_equal(a, np.swapaxes(a, -1, -2))
    if name in ("box1", "box2"):  # exact zeros where the full tree has noise
        nb = 2 * L + 1
        odd = np.array([((m // nb) in (2, 4)) ^ ((m % nb) in (2, 4)) for m in range(M)])
        mask = odd[:, None] ^ odd[None, :]
        assert (a[..., mask] == 0.0).all() and (np.abs(b[..., mask]) <= 1e-13 * l1[..., 0]).all()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("kind", [0, 1, 2])
def test_integrand_kinds_and_both_kernels(P, kind, layout):
    (a, _, sa, ra), (b, _, sb, rb) = both(P, W.ff_box(1), 1, 1e-7, kind=kind, eval_layout=layout)
    assert ra == P.OK and rb == P.OK
    assert (np.abs(a - b) <= 2e-7 * np.abs(b).sum(axis=(-1, -2), keepdims=True)).all()


@pytest.mark.parametrize("budget", [16, 17, 64, 100])
def test_budgets_of_odd_sizes(P, budget):
    """a container never holds more than max_regions leaves of the whole zone"""
    with P.Context(max_regions=budget) as c:
        out, _, st, rc = c.integrate(ROWS, Q, W.ff_box(1), 1, rtol=1e-9)
    assert rc == P.ENOCONV and st["not_converged"] == st["containers"] == 20
    assert st["regions"] <= 20 * budget and np.isfinite(out).all()


def test_even_and_general_seed_models(P):
    """an even model starts both images from one tree, any other the whole zone"""
    from paid_1610_09991_amd import seed_model as SM
    w, _ = SM.load()
    for model in (SM.even(w), w):
        (a, _, sa, ra), (b, _, sb, rb) = both(P, W.ff_box(1), 1, 1e-6, model=model)
        assert ra == P.OK and rb == P.OK and sa["seeded"] == sb["seeded"] == 20
        assert (np.abs(a - b) <= 2e-6 * np.abs(b).sum(axis=(-1, -2), keepdims=True)).all()
        assert abs(sa["regions"] - sb["regions"]) <= 0.02 * sb["regions"]
        if model is w:
            assert np.array_equal(a, b) and sa["regions"] == sb["regions"]


def test_labels_count_both_images(P):
    n = len(ROWS) * len(Q) * 2
    x, y = np.zeros((n, 7), dtype=np.float32), np.zeros((n, 256), dtype=np.float32)
    with P.Context(max_regions=1 << 16) as c:
        c.set_label_output(x, y)
        _, _, st, rc = c.integrate(ROWS, Q, W.ff_box(1), 1, rtol=1e-6)
    assert rc == P.OK
    leaves = np.sum(np.exp2(y.astype(np.float64)) - 1.0)
    assert abs(leaves - st["regions"]) <= 1e-5 * st["regions"]
    assert np.array_equal(y, y[:, ::-1])


def test_batch_of_two_splits_one_pair_a_round(P):
    """batch_max 2: one stored leaf and its image a round"""
    with P.Context(max_regions=1 << 12, batch=1, batch_max=2) as c:
        a, _, st, rc = c.integrate(ROWS[1:], Q[:1], W.ff_box(1), 1, rtol=1e-3)
    with P.Context(max_regions=1 << 12) as c:
        b, _, _, _ = c.integrate(ROWS[1:], Q[:1], W.ff_box(1), 1, rtol=1e-6)
    assert rc == P.OK and st["rounds"] >= (st["splits"] - 2) // 2
    assert (np.abs(a - b) <= 1.1e-3 * np.abs(b).sum(axis=(-1, -2), keepdims=True)).all()
