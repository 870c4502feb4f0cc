"""Plans kept with room for many more segments than they hold, as the server
keeps them: values of requests around the sizes where a wave's part of an item
begins or stays empty, near the start of a stream and far into it, against the
oracle, with fewer and more items than the waves that share them."""
import random

import numpy as np
import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx

pytestmark = pytest.mark.gpu

P = 2048


@pytest.mark.parametrize("n", (1, 100, 1000, 2049, 4097, 9000))
@pytest.mark.parametrize("lanes", (16, 64))
def test_kept_plan_with_large_capacity(n, lanes):
    rng = random.Random(n + lanes)
    counts = [min(rng.choice((1, 12 * lanes, 24 * lanes + 5, 48 * lanes - 1, 48 * lanes + 1, 96 * lanes, 12 * lanes * 9)), 12000 if n < 5000 else 400)
              for _ in range(n)]
    starts = [rng.choice((0, 7, 12 * 65535 + 3, 12 * (1 << 33) + 5)) for _ in range(n)]
    states = rlx.new_states(64)
    rlx.init_streams(states, P, id0=1)
    req = rlx.requests_array([k % 64 for k in range(n)], starts, counts, P)
    plan = rlx.Plan(rlx.requests_array(np.zeros(0, dtype=np.uint64), 0, np.zeros(0, dtype=np.uint64), P),
                    lanes=lanes, seg_blocks=8192, capacity_segments=87381)
    plan.update(req)
    out = torch.full((plan.extent + 1,), -1, dtype=torch.int64, device="cuda")
    u = plan.generate_u64(states, out).cpu().numpy()
    assert rlx.check_errors() == 0 and u[-1] == -1 and (u[:-1] >= 0).all()
    for k in sorted({0, n - 1} | {rng.randrange(n) for _ in range(40)}):
        o = int(req[k]["out_offset"])
        assert u[o:o + counts[k]].tolist() == O.window(O.seed(1 + k % 64, P), P, starts[k], counts[k]), k
