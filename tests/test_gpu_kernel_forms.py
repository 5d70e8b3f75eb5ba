"""The frequency-summed kernel in both forms that the evaluation kernels use:
value rows with close rows for close pairs (eval_layout 0), and close rows alone
(eval_layout 1, the one-wave kernel's), against the oracle on the energy pairs
and within the bar of the other kernel test (2e-12 of the local scale)."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import adversarial

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,Om", [(0.005, 0.01), (0.01, 10.0), (0.1, 1.0), (2.0, 0.3)])
def test_both_forms_match_the_oracle(T, Om):
    import paid_1610_09991_amd as P
    pts = adversarial(Om, T, 5.95)
    a, b = (np.array(x) for x in zip(*pts))
    got = {}
    for layout in (0, 1):
        with P.Context(eval_layout=layout) as c:
            for ch, och in ((P.PH, O.PH), (P.PP, O.PP)):
                got[layout, ch] = g = c.kernel((1.0, -0.25, -0.95, T, Om), a, b, ch)
                for x, y, v in zip(a, b, g):
                    ref = O.kernel(x, y, Om, T, och)
                    loc = abs(O.kernel(abs(x) + 0.5 * T, abs(x) + 0.5 * T, Om, T, O.PH))
                    assert abs(v - ref) <= 2e-12 * max(abs(ref), loc), (layout, ch, x, y, v, ref)
    # two forms: far pairs round differently somewhere
    assert any(not np.array_equal(got[0, ch], got[1, ch]) for ch in (P.PH, P.PP))
