"""Batched launch: waves that share an item, items in groups of one level, and
the lane start-up of segments far into a stream.  Values of whole requests (or
of their windows) against the oracle: requests around the sizes where a part
of an item begins or stays empty, starts whose first 16-bit digit wraps inside
a segment's lanes, plans with fewer and with more items than the waves that
are shared out, and an update from one to the other under one launch shape."""
import random

import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx
from rlx_util import records_to_tensor

pytestmark = pytest.mark.gpu

LEVELS = (24, 404, 2048)


def run(plan_args, reqs, n_states, picks=None):
    """reqs: (state, start, count, p); checks the requests in picks (all)."""
    st = records_to_tensor([(O.seed(7 * i, LEVELS[i % 3]), 0, LEVELS[i % 3]) for i in range(n_states)])
    req = rlx.requests_array(*(list(v) for v in zip(*reqs)))
    plan = rlx.Plan(req, **plan_args)
    out = torch.full((plan.extent + 1,), -1, dtype=torch.int64, device="cuda")
    u = plan.generate_u64(st, out).cpu().numpy()
    assert rlx.check_errors() == 0 and u[-1] == -1
    for k in picks if picks is not None else range(len(reqs)):
        s, start, count, p = reqs[k]
        o = int(req[k]["out_offset"])
        assert u[o:o + count].tolist() == O.window(O.seed(7 * s, p), p, start, count), (k, reqs[k])
    return plan, st, out


@pytest.mark.parametrize("lanes", (1, 16, 32, 64))
def test_parts_of_items(lanes):
    # iterations of an item: 1, 2, 3 (parts stay empty), around 64 waves' worth
    reqs = []
    for i, its in enumerate((1, 2, 3, 4, 5, 127, 128, 129, 130)):
        for d in (-1, 0, 1):
            count = min(12 * lanes * its, 40000) + d
            reqs.append((len(reqs) % 30, (11 * i) % 37, count, LEVELS[(len(reqs) % 30) % 3]))
    run(dict(lanes=lanes, seg_blocks=4096), reqs, 30)


@pytest.mark.parametrize("lanes", (8, 32, 64))
def test_starts_across_window_digits(lanes):
    starts = [12 * b + f for b in (65535, 65536, 65536 - lanes // 2, 131072 - 1, (1 << 32) - 3, (1 << 48) - lanes)
              for f in (0, 7)]
    reqs = [(i, s, 12 * lanes * 2 + 5, LEVELS[i % 3]) for i, s in enumerate(starts)]
    run(dict(lanes=lanes, seg_blocks=64), reqs, len(reqs))


def test_more_items_than_shared_waves_and_update():
    rng = random.Random(8)
    n = 9000
    reqs = [(i % 300, rng.randrange(100), rng.randrange(1, 40), LEVELS[(i % 300) % 3]) for i in range(n)]
    plan, st, out = run(dict(lanes=64, seg_blocks=4096), reqs, 300, rng.sample(range(n), 300))
    # the same plan with a few longer requests: the spare waves share them
    few = [(i, 5 * i, 4000 + 700 * i, LEVELS[i % 3]) for i in range(7)]
    req = rlx.requests_array(*(list(v) for v in zip(*few)))
    plan.update(req)
    u = plan.generate_u64(st, out).cpu().numpy()
    for k, (s, start, count, p) in enumerate(few):
        o = int(req[k]["out_offset"])
        assert u[o:o + count].tolist() == O.window(O.seed(7 * s, p), p, start, count), k
    assert plan.info()["items"] == 7


# header, items and segments up to 1 MiB (about 16 000 requests) go up through
# a kernel, more through the copy engine; updates queue behind launches
@pytest.mark.parametrize("first,second", ((1, 16000), (15900, 17000), (17000, 3), (16300, 16400)))
def test_update_sizes(first, second):
    rng = random.Random(first)
    sets = [[(i % 40, rng.randrange(50), rng.randrange(1, 30), LEVELS[(i % 40) % 3]) for i in range(n)]
            for n in (first, second)]
    reqs = [rlx.requests_array(*(list(v) for v in zip(*s))) for s in sets]
    st = records_to_tensor([(O.seed(7 * i, LEVELS[i % 3]), 0, LEVELS[i % 3]) for i in range(40)])
    plan = rlx.Plan(reqs[0], capacity_segments=20000, lanes=64, seg_blocks=4096)
    outs = []
    for req in (reqs[0], reqs[1], reqs[0]):
        plan.update(req)
        outs.append(plan.generate_u64(st, torch.empty(plan.extent, dtype=torch.int64, device="cuda")))
    assert rlx.check_errors() == 0
    for (rs, req), out in zip(zip((sets[0], sets[1], sets[0]), (reqs[0], reqs[1], reqs[0])), outs):
        u = out.cpu().numpy()
        picks = {0, len(rs) - 1} | {rng.randrange(len(rs)) for _ in range(60)}
        for k in picks:
            s, start, count, p = rs[k]
            o = int(req[k]["out_offset"])
            assert u[o:o + count].tolist() == O.window(O.seed(7 * s, p), p, start, count), k
