"""Lane start-up and generator step of the generate kernels on the matrix cores
(include/rlx_mfma.hpp): X_l = A_p^l X_0 as a contraction with the Toeplitz
matrix of X_0's balanced digits (32 or more lanes per record), and the step
with contiguous output halves.  Values and records are compared with the
oracle for states at the edges of the digit form (bytes and words where the
balancing carries, the ends of [0, m), single bytes) and for states whose
product ends where a carry or borrow of the fold runs on (the branch that
settles them); for one lane per record up to several waves per record; and
next to records that are rejected."""
import random

import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx
from rlx_util import records_to_tensor, tensor_to_records

pytestmark = pytest.mark.gpu


def edge_states():
    m = O.M
    fill = lambda b: sum(b << (8 * i) for i in range(72))
    runs = [((1 << (32 * hi)) - (1 << (32 * lo))) & fill(0x7F) for lo, hi in ((0, 1), (0, 17), (3, 9), (1, 18))]
    xs = [0, 1, m - 1, m - 2, 2 ** 240, 2 ** 240 - 1, 2 ** 575, 2 ** 576 - 2 ** 241,
          fill(0x7F), fill(0x7F) + 1, fill(0x80), fill(0x80) - 1, fill(0x81), fill(0xFF) % m]
    # a run of propagating words with and without a carry into it
    xs += [r + d for r in runs for d in (0, 1, 0x7F7F7F80 << 32)]
    xs += [1 << (8 * i) for i in range(0, 72, 5)] + [0x80 << (8 * i) for i in range(0, 71, 7)]
    rng = random.Random(5)
    xs += [rng.randrange(m) for _ in range(20)]
    return [x % m for x in xs]


@pytest.fixture(autouse=True)
def lanes_reset():
    yield
    rlx.set_lanes_per_stream(0)


def settled_states(p, steps):
    """States X whose product A_p^steps X has words where the folding's sums
    end: a borrow past word 1, a carry past word 8, the low half's carry past
    word 10 (either sign), a top word of all ones."""
    m, rng = O.M, random.Random(steps)
    inv = pow(O.multiplier(p), -steps, m)
    ones = 0xFFFFFFFF

    def with_words(words):
        x = rng.randrange(m)
        for k, v in words.items():
            x = x & ~(ones << (32 * k)) | v << (32 * k)
        return x % m
    out = []
    for small in (0, 1, 5, 200, 4000):
        out += [with_words({0: ones - small, 1: ones}), with_words({0: ones - small, 1: ones, 2: ones}),
                with_words({7: small << 16, 8: 0}), with_words({7: small << 16, 8: 0, 9: 0}),
                with_words({9: small, 10: 0}), with_words({9: small, 10: 0, 11: 0}),
                with_words({9: ones - small, 10: ones}), with_words({9: ones - small, 10: ones, 11: ones}),
                with_words({17: ones}), m - 1 - small, small]
    return [x * inv % m for x in out]


@pytest.mark.parametrize("G", (1, 2, 16, 32, 64))
@pytest.mark.parametrize("general", (False, True))
def test_step_settles_carries(G, general):
    p = 2048
    xs = settled_states(p, G) + settled_states(p, 1) + settled_states(p, 7)
    recs = [(x, (5 * i) % 12, p) for i, x in enumerate(xs)]
    count = 24 * G + 13
    st = records_to_tensor(recs)
    rlx.set_lanes_per_stream(G)
    gen = rlx.test_generate_u64_general if general else rlx.generate_u64
    u, after = gen(st, count, p).cpu().numpy(), tensor_to_records(st)
    for i, (x, pos, _) in enumerate(recs):
        vals, x2, pos2 = O.draws(x, pos, p, count)
        assert u[i].tolist() == vals and after[i] == (x2, pos2, p), i


@pytest.mark.parametrize("G", (1, 2, 16, 32, 64, 128))
@pytest.mark.parametrize("p", (24, 2048))
def test_edge_states(p, G):
    recs = [(x, (7 * i) % 12, p) for i, x in enumerate(edge_states())]
    count = 12 * G + 30     # every lane's first block, some lanes' second
    st = records_to_tensor(recs)
    rlx.set_lanes_per_stream(G)
    u = rlx.generate_u64(st, count, p).cpu().numpy()
    assert rlx.check_errors() == 0
    after = tensor_to_records(st)
    for i, (x, pos, _) in enumerate(recs):
        vals, x2, pos2 = O.draws(x, pos, p, count)
        assert u[i].tolist() == vals, (i, hex(x))
        assert after[i] == (x2, pos2, p), i


@pytest.mark.parametrize("G", (32, 64))
def test_shared_start_next_to_rejected_records(G):
    p, count = 404, 500
    m = O.M
    good = [(O.seed(i, p), i % 12, p) for i in range(9)]
    recs = list(good)
    recs[1] = (m, 0, p)                  # X >= m, smallest
    recs[4] = (2 ** 576 - 1, 3, p)       # and largest
    recs[5] = (good[5][0], 12, p)        # pos > 11
    recs[6] = (good[6][0], 0, p + 1)     # another level
    recs[7] = (m - 1, 11, p)             # the largest state that is one
    st = records_to_tensor(recs)
    rlx.set_lanes_per_stream(G)
    out = torch.full((len(recs), count), -1, dtype=torch.int64, device="cuda")
    rlx.generate_u64(st, count, p, out=out)
    assert rlx.check_errors() == 0x7     # BAD_P | BAD_POS | BAD_X
    u, after = out.cpu().numpy(), tensor_to_records(st)
    for i, (x, pos, q) in enumerate(recs):
        if i in (1, 4, 5, 6):
            assert (u[i] == -1).all() and after[i] == (x, pos, q), i
        else:
            vals, x2, pos2 = O.draws(x, pos, p, count)
            assert u[i].tolist() == vals and after[i] == (x2, pos2, p), i


# records of several levels around one round of the 32-lane kernel's waves,
# where calls that pick their own lanes go from 32 to 64 and back
@pytest.mark.parametrize("n", (6144, 6145, 9216, 9217))
@pytest.mark.parametrize("count", (370, 397))
def test_levels_around_one_round(n, count):
    levels = (24, 404, 2048)
    rng = random.Random(n + count)
    for p in levels:
        rlx.prepare(p)
    st = rlx.new_states(n)
    for k, p in enumerate(levels):
        st[k::3] = rlx.init_streams(rlx.new_states(st[k::3].shape[0]), p, id0=1000 * k)
    u = rlx.generate_u64(st, count, rlx.P_RECORD)
    assert rlx.check_errors() == 0
    for i in [0, 1, 2, n - 1] + rng.sample(range(n), 20):
        p = levels[i % 3]
        x = O.seed(1000 * (i % 3) + i // 3, p)
        assert u[i].tolist() == O.window(x, p, 0, count), i
        assert tensor_to_records(st[i:i + 1]) == [O.state_at(x, p, count) + (p,)], i
