"""The contraction with the couplings' own arrays as outputs, through the C ABI
on device memory: one and two column tiles, few momenta and many.  The same
sums in the same order as into separate arrays: equal bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 9, 16, 17, 25, 32])
@pytest.mark.parametrize("n_l", [1, 3, 2000])
def test_outputs_over_the_couplings(M, n_l):
    import torch

    import paid_1610_09991_amd as P
    rng = np.random.default_rng(100 * M + n_l)
    dev = dict(dtype=torch.float64, device="cuda:0")
    chi = torch.tensor(rng.normal(size=(n_l, 2, M, M)), **dev)
    V = [torch.tensor(rng.normal(size=(n_l, M, M)), **dev) for _ in range(3)]
    ptr = lambda a: a.data_ptr()
    with P.Context() as c:
        ref = c.contract(chi, *V)
        for which in ([0], [1], [2], [0, 1, 2]):
            a = [v.clone() for v in V]
            out = [a[i] if i in which else torch.empty_like(V[i]) for i in range(3)]
            torch.cuda.synchronize()
            rc = P.lib().paid_contract(c.h, n_l, M, *[P.C.c_void_p(ptr(x)) for x in (chi, *a, *out)])
            assert rc == P.OK
            assert all(torch.equal(o, r) for o, r in zip(out, ref)), which
