"""The planner gives the shapes of the GPU tests the variants that those tests name."""
import pytest

from tests.x3_shapes import PLANS, VARIANTS, plan


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
