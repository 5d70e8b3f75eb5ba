"""The automatic number of resident containers leaves room for the buffers of a
round.  A card filled up to 16 GiB, one form factor and up to 69,600 splits a
round and container, a leaf budget at which the pool's share (0.55 of what is
free) and the round buffers' share (0.35) bind together: all of it has to fit, and
the containers beyond the first ones are taken in turn."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_round_buffers_fit_beside_the_pool():
    import torch

    import paid_1610_09991_amd as P
    q = W.q_grid(64)
    ref = P.Context(max_regions=1 << 12, pool_gib=1.0)
    want = ref.integrate([[1.0, -0.25, -0.95, 0.3, 1.0]], q, W.ff_box(0), 0, P.PH, rtol=1e-2)
    ref.close()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    filler = torch.empty(free - (16 << 30), dtype=torch.uint8, device="cuda:0")
    try:
        with P.Context(max_regions=2 * 109_375, batch_max=2 * 69_600) as c:
            slots = 3500
            for _ in range(3):  # no later call asks for a larger pool
                out, _, st, rc = c.integrate([[1.0, -0.25, -0.95, 0.3, 1.0]], q, W.ff_box(0), 0, P.PH, rtol=1e-2)
                left, _ = torch.cuda.mem_get_info()
                assert rc == P.OK and st["containers"] == 4096
                assert 1000 < st["max_active"] <= slots, (st["max_active"], slots)
                slots = st["max_active"]
                assert left > 0.08 * (16 << 30), left
    finally:
        del filler
        torch.cuda.empty_cache()
    assert np.array_equal(out, want[0])
