"""Skips of records that pass through LDS: counts around a wave and a block,
one offset for all and one each (where other lanes, of other waves, may handle
a record), and refused records, which stay as they are between others."""
import random

import numpy as np
import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx
from rlx_util import records_to_tensor, tensor_to_records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 63, 64, 65, 255, 256, 257, 449))
@pytest.mark.parametrize("each", (False, True))
def test_skips_around_blocks(n, each):
    rng = random.Random(n)
    p = 2048
    recs = [(O.seed(i, p), rng.randrange(12), p) for i in range(n)]
    refused = {i for i in range(n) if i % 37 == 5}
    for i in refused:  # another level, a state that is not reduced, a position past the block
        x, pos, _ = recs[i]
        recs[i] = ((x, pos, 24), (O.M, pos, p), (x, 12, p))[i % 3]
    by = [rng.getrandbits(rng.randrange(0, 65)) for _ in range(n)] if each else [3 * n + 70001] * n
    arg = torch.from_numpy(np.array(by, dtype=np.uint64).view(np.int64)).cuda() if each else by[0]
    for values in (False, True):
        guard = records_to_tensor(recs + [(1, 0, p)] * 3)
        (rlx.skip_values if values else rlx.skip)(guard[:n], arg, p)
        assert (rlx.check_errors() != 0) == bool(refused)
        got = tensor_to_records(guard)
        assert got[n:] == [(1, 0, p)] * 3
        for i in range(n):
            x, pos, q = recs[i]
            if i not in refused:
                steps, pos = divmod(pos + by[i], 12) if values else (by[i], pos)
                x = O.skip(x, steps, p)
            assert got[i] == (x, pos, q), (i, values)
