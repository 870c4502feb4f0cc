"""rlx_call_lanes: the lanes per record that calls take (no GPU needed).  Powers
of two within the launch limits for every kind of draw, forced lanes and the
vector-ALU step included; the shape of the test of records that span many
waves does span them."""
import pytest

import paper_2106_02504_amd as rlx

LEVELS = ("levels", "levels_normal")


@pytest.fixture(autouse=True)
def reset():
    yield
    rlx.set_lanes_per_stream(0)
    rlx.set_step_kernel(rlx.STEP_MFMA)


@pytest.mark.parametrize("kind", tuple(rlx.DRAW_KINDS))
def test_call_lanes(kind):
    for n in (1, 3, 64, 100, 5000, 1 << 16, 100000, (1 << 21) + 1, 1 << 30):
        for count in (1, 11, 12, 24, 100, 1000, 1 << 16, 1 << 20, 1 << 24, 1 << 35):
            g = rlx.call_lanes(kind, n, count)
            assert g & (g - 1) == 0 and 1 <= g <= (64 if kind in LEVELS else 65536)
            assert g == 1 or n * g <= 1 << 21
            assert g <= 2 * (count // 11 + 1)
            rlx.set_step_kernel(rlx.STEP_VALU)
            nominal = rlx.lanes_per_stream(n, count)
            assert rlx.call_lanes(kind, n, count) == (min(nominal, 64) if kind in LEVELS else nominal)
            rlx.set_step_kernel(rlx.STEP_MFMA)
    for forced in (1, 16, 64, 256, 65536):
        rlx.set_lanes_per_stream(forced)
        assert rlx.call_lanes(kind, 5000, 1000) == (min(forced, 64) if kind in LEVELS else forced)


def test_shapes_that_other_tests_mean():
    assert rlx.call_lanes("uniform", 16, 1 << 24) > 64 and rlx.call_lanes("legacy", 16, 1 << 24) > 64
    assert rlx.call_lanes("uniform", 65536, 4096) == 32   # the kernel that the profiles are of


def test_unknown_kinds():
    lib = rlx.lib()
    assert lib.rlx_call_lanes(-1, 5, 10) == 0 and lib.rlx_call_lanes(6, 5, 10) == 0
