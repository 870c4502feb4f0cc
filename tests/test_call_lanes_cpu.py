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


# shapes where the estimate without the waves per SIMD, or with the uniform
# draw's costs for all, took far too few or too many lanes: the least and the
# most lanes within 5% of the best measured
@pytest.mark.parametrize("kind,n,count,least,most", (
    ("uniform", 2100, 50000, 512, 1024), ("uniform", 4200, 25000, 256, 512), ("uniform", 8192, 10000, 64, 128),
    ("normal", 10000, 4096, 32, 32), ("normal", 25000, 4096, 16, 32),
    ("legacy", 2100, 50000, 256, 1024), ("traced", 32768, 30, 2, 4), ("legacy", 500000, 30, 2, 4),
    ("levels", 8192, 1000, 32, 32), ("levels", 6500, 4000, 32, 64), ("levels", 65536, 4096, 32, 64)))
def test_picks(kind, n, count, least, most):
    assert least <= rlx.call_lanes(kind, n, count) <= most


def test_unknown_kinds():
    lib = rlx.lib()
    assert lib.rlx_call_lanes(-1, 5, 10) == 0 and lib.rlx_call_lanes(6, 5, 10) == 0
