"""Register budget of the kernels for records of several levels, from the
compiler's resource report as in test_kernel_resources: four waves per SIMD
and no spills with 32 lanes per record, where half-waves hold one record each
and the matrix-core step has two multipliers; four waves with fewer lanes and
next to no spills."""
import pytest

from test_kernel_resources import OUT_KINDS, resources  # noqa: F401  (fixture)


def levels_kernel(table, kind, lgs):
    hits = [v for k, v in table.items() if f"k_generate_levelsILN3rlx3OutE{OUT_KINDS[kind]}ELi{lgs}E" in k]
    assert len(hits) == 1, (kind, lgs)
    return hits[0]


@pytest.mark.parametrize("kind", tuple(OUT_KINDS))
def test_levels_kernels(resources, kind):  # noqa: F811
    for lgs in range(1, 6):
        r = levels_kernel(resources, kind, lgs)
        assert r["Occupancy"] == 4, (lgs, r)
        assert r["ScratchSize"] <= (0 if lgs == 5 else 16), (lgs, r)
