"""The ring walk of three to eight learners, at the edges of where it is used and with tables that are not one ring.  Every element against
the oracle."""
import pytest

import test_gpu_short_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
psgd = test_gpu_short_rows.psgd


# learners times column groups: 24 000 per compute unit with the distance, 100 000 without (256 compute units)
@pytest.mark.parametrize("n,d,deg,gkind,extra", [
    (3, 8_191_996, 3, "f32", None), (3, 8_192_001, 3, "bf16", (1, 2, 3)), (4, 6_143_997, 3, "bf16", None), (4, 6_144_002, 3, "f32", None),
    (5, 4_915_201, 3, "f32", (3, 1, 2)), (6, 4_096_003, 3, "bf16", None), (6, 17_066_668, 3, "f32", None), (7, 3_510_859, 3, "f32", None),
    (8, 3_071_996, 3, "bf16", None), (8, 12_799_997, 3, "f32", (1, 2, 3)),
    (3, 8_192_004, -3, "f32", None), (4, 6_144_001, -3, "bf16", (1, 2, 3)), (5, 4_915_204, -3, "bf16", None), (7, 3_510_861, -3, "f32", None),
    (8, 12_800_004, -3, "f32", None)])
def test_ring_walk_of_few_learners(psgd, n, d, deg, gkind, extra):
    test_gpu_short_rows.test_short_rows_every_element(psgd, n, d, deg, gkind, extra)
