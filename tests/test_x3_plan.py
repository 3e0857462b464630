"""The planner gives the shapes of the GPU tests the variants that those tests name."""
import pytest

from tests.x3_shapes import OLDER, PLANS, VARIANTS, plan


@pytest.mark.parametrize("variant, t, dtype, halo", PLANS)
def test_shape_is_planned_for_its_variant(variant, t, dtype, halo):
    p, taken = plan(t, dtype)
    assert taken in (1, 2) and (p.variant, p.halo) == (variant, halo)
    assert p.tiles >= 2 * p.splits                                  # several tiles to a workgroup
    assert p.splits == 1 or p.tiles % p.splits                      # of different numbers
    SH = 32 if p.ktiles == -(-t[4] // 32) else 16
    assert t[4] % SH or t[4] % 64                                   # a ragged last tile of output channels


def test_every_variant_has_a_shape():
    assert {v for v, *_ in PLANS} == set(range(VARIANTS))


@pytest.mark.parametrize("t, dtype", OLDER)
def test_shape_stays_with_the_older_forms(t, dtype):
    assert plan(t, dtype)[1] == 0


def test_whole_bf16_rows_are_not_staged_element_by_element():
    """Two-byte loads, one column at a time: 64 -> 64 @ 56x56, stride 2, N = 128 took 162 us that way (105 widened to fp32),
    32 -> 32 @ 64x64, N = 87, 113 (93)."""
    for t in ((128, 64, 56, 56, 64, 3, 3, 2, 2, 1, 1), (87, 32, 64, 64, 32, 3, 3, 1, 1, 1, 1)):
        assert plan(t, "bf16")[0].variant in (12, 13, 15, 17)
