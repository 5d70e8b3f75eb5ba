"""A scan of more parameter rows than one launch of the table kernels may have
threads for (84 workgroups of 256 a row at T = 0.01: 2^32 threads at 199,729
rows).  The tables of the rows are then built by several launches; a row's
integrals are those of a call of few rows, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_two_hundred_thousand_rows():
    import paid_1610_09991_amd as P
    n = 205_000
    rng = np.random.default_rng(4)
    rows = np.stack([np.ones(n), rng.uniform(-0.35, 0.0, n), rng.uniform(-1.2, 0.0, n), np.full(n, 0.01),
                     np.exp(rng.uniform(np.log(0.5), np.log(10.0), n))], axis=1)
    rows[7, 3] = 0.3  # a shorter table between them
    pick = np.array([0, 1, 6, 7, 8, 99_863, 99_864, 99_865, 199_728, 199_729, n - 1])
    args = ([[2.88, 0.26]], np.ones((1, 1)), 0, P.PH)
    with P.Context(max_regions=256, pool_gib=1.0) as c:
        out, _, st, _ = c.integrate(rows, *args, rtol=0.1)
    with P.Context(max_regions=256, pool_gib=1.0) as c:
        ref, _, _, rc = c.integrate(rows[pick], *args, rtol=0.1)
    assert st["containers"] == n and rc == P.OK
    assert np.isfinite(out).all() and (out != 0.0).all()
    assert np.array_equal(out[pick], ref)
