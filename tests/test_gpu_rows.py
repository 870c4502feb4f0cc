"""One lane per record (many records, few values each): values and records
against the oracle around the sizes where the kernel changes its way of
storing (one step's 12 values, two steps' 24, odd and even counts and
positions, rows kept whole or not), waves that are not full, rejected records
among good ones, and outputs on 8-byte boundaries; the other output kinds
against the same draws with two lanes per record."""
import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx
from rlx_util import records_to_tensor, tensor_to_records

pytestmark = pytest.mark.gpu

P = 404


@pytest.fixture(autouse=True)
def one_lane():
    rlx.set_lanes_per_stream(1)
    yield
    rlx.set_lanes_per_stream(0)


def records(n, start):
    """n records at position `start`, or at mixed positions for None."""
    return [(O.seed(3 * i, P), (5 * i) % 12 if start is None else start, P) for i in range(n)]


def check(recs, u, st, count, skip=()):
    after = tensor_to_records(st)
    for i, (x, pos, p) in enumerate(recs):
        if i in skip:
            assert (u[i] == -1).all() and after[i] == recs[i], i
        else:
            vals, x2, pos2 = O.draws(x, pos, p, count)
            assert u[i].tolist() == vals, i
            assert after[i] == (x2, pos2, p), i


@pytest.mark.parametrize("count", (1, 2, 7, 11, 12, 13, 14, 23, 24, 25, 36, 37, 61))
@pytest.mark.parametrize("start", (0, 1, 4, 11, None))
def test_rows(count, start):
    recs = records(130, start)
    st = records_to_tensor(recs)
    check(recs, rlx.generate_u64(st, count, P).cpu().numpy(), st, count)
    assert rlx.check_errors() == 0


@pytest.mark.parametrize("n", (1, 63, 64, 65, 257))
@pytest.mark.parametrize("count", (12, 24, 26))
def test_rows_partial_waves(n, count):
    recs = records(n, 0)
    st = records_to_tensor(recs)
    check(recs, rlx.generate_u64(st, count, P).cpu().numpy(), st, count)


@pytest.mark.parametrize("count", (11, 24, 31))
def test_rows_rejected_records(count):
    recs = records(140, 2)
    bad = (0, 17, 64, 139)
    for k, i in enumerate(bad):
        recs[i] = ((O.M, 2, P), (recs[i][0], 12, P), (recs[i][0], 2, P + 1), (2 ** 576 - 1, 0, P))[k]
    st = records_to_tensor(recs)
    out = torch.full((len(recs), count), -1, dtype=torch.int64, device="cuda")
    rlx.generate_u64(st, count, P, out=out)
    assert rlx.check_errors() == 0x7
    check(recs, out.cpu().numpy(), st, count, skip=bad)


@pytest.mark.parametrize("count", (12, 24, 40))
def test_rows_output_on_8_byte_boundary(count):
    recs = records(70, 0)
    st = records_to_tensor(recs)
    buf = torch.full((1 + 70 * count + 1,), -1, dtype=torch.int64, device="cuda")
    rlx.generate_u64(st, count, P, out=buf[1:-1].view(70, count))
    check(recs, buf[1:-1].view(70, count).cpu().numpy(), st, count)
    assert int(buf[0]) == -1 and int(buf[-1]) == -1


@pytest.mark.parametrize("kind", ("f64", "f32", "normal_f64"))
@pytest.mark.parametrize("start", (0, 3, None))
def test_rows_other_kinds(kind, start):
    gen = getattr(rlx, "generate_" + kind)
    for count in (12, 24, 50):
        a = records_to_tensor(records(100, start))
        b = a.clone()
        rlx.set_lanes_per_stream(1)
        x = gen(a, count, P)
        rlx.set_lanes_per_stream(2)
        y = gen(b, count, P)
        assert torch.equal(x, y) and torch.equal(a, b), count
