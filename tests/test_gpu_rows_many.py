"""One lane per record with enough records for the kernel that passes records
and rows through LDS (below that the ordinary kernel runs): every output kind,
records at one position, an odd one and mixed ones, refused records, outputs on
8-byte boundaries and numbers of records on both sides of where a wave's mixed
rows are stored joined; against the same draws with two lanes per record, which
other tests compare with the oracle, and single records with the oracle."""
import statistics

import pytest
import torch

import oracle as O
import paper_2106_02504_amd as rlx
from rlx_util import tensor_to_records

pytestmark = pytest.mark.gpu

P = 794
KINDS = {"f64": (rlx.generate_f64, torch.float64, 1), "u64": (rlx.generate_u64, torch.int64, 1),
         "f32": (rlx.generate_f32, torch.float32, 2), "normal": (rlx.generate_normal_f64, torch.float64, 1)}


@pytest.fixture(autouse=True)
def lanes_reset():
    yield
    rlx.set_lanes_per_stream(0)


def records(n, start):
    st = rlx.new_states(n)
    rlx.init_streams(st, P, id0=1)
    if start is None:
        rlx.skip_values(st, (torch.arange(n, dtype=torch.int64, device="cuda") * 7) % 12, P)
    else:
        rlx.skip_values(st, start, P)
    return st


def draws(kind, st, count, lanes, offset):
    """(outputs with what lies before and after them, records)"""
    call, dtype, per = KINDS[kind]
    n = st.shape[0]
    flat = torch.full((n * count * per + 64,), 7, dtype=dtype, device="cuda")
    lo = 16 + offset * per
    out = flat[lo:lo + n * count * per].view(n, count * per)
    rlx.set_lanes_per_stream(lanes)
    call(st, count * per, P, out=out)
    return flat, st


@pytest.mark.parametrize("n", (32768 + 65, 49152 + 1, 131072 + 130))
@pytest.mark.parametrize("count", (1, 6, 11, 12, 13, 24, 25, 37))
@pytest.mark.parametrize("start", (0, 5, None))
def test_rows_of_many_records(n, count, start):
    for kind, offset in (("u64", 0), ("f64", 1), ("f32", 0)):
        st = records(n, start)
        first = tensor_to_records(st[:70])
        a = draws(kind, st.clone(), count, 1, offset)
        b = draws(kind, st.clone(), count, 2, offset)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), kind
        if kind == "u64":
            rows = a[0][16:16 + n * count].view(n, count)
            for i in (0, 1, 63, 64, 69):
                x, pos, p = first[i]
                assert rows[i].tolist() == O.draws(x, pos, p, count)[0], i
    assert rlx.check_errors() == 0


@pytest.mark.parametrize("n,count", ((32768 + 65, 12), (32768 + 65, 25), (65536 + 65, 25),
                                     (262144 + 1, 1), (262144 + 1, 5), (262144 + 1, 7)))
@pytest.mark.parametrize("start", (0, None))
def test_normal_rows(n, count, start):
    st = records(n, start)
    a, b = (draws("normal", st.clone(), count, lanes, 0) for lanes in (1, 2))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("count", (5, 12, 20))
@pytest.mark.parametrize("start", (0, None))
def test_refused_records_between_others(count, start):
    st = records(32768 + 65, start)
    bad = torch.arange(st.shape[0], device="cuda") % 29 == 3
    st[bad, 9] += 1 << 32  # another level
    a, b = (draws("u64", st.clone(), count, lanes, 0) for lanes in (1, 2))
    assert rlx.check_errors() != 0
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert torch.equal(a[1][bad], st[bad])


def test_few_records_at_mixed_positions_cost_no_more():
    # (27 us against 17 when their values left as joined rows)
    def us(start):
        st = records(1000, start)
        out = torch.empty((1000, 96), dtype=torch.float64, device="cuda")
        rlx.set_lanes_per_stream(1)
        times = []
        for _ in range(8):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(20):
                rlx.generate_f64(st, 96, P, out=out)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1) * 50)
        return statistics.median(times[2:])
    assert us(None) < 1.35 * us(0)


@pytest.mark.parametrize("count,offset", ((12, 2), (13, 6), (24, 2), (24, 8)))
def test_whole_rows_off_a_line(count, offset):
    # outputs on 16-byte boundaries inside a line
    st = records(49152 + 1, 0)
    a, b = (draws("f64", st.clone(), count, lanes, offset) for lanes in (1, 2))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
