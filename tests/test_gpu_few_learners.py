"""The ring walk of three to eight learners, at the edges of where it is used and with tables that are not one ring, the next gradients of
the delay-by-one schedule from the short-row kernel in each of its forms, global averaging of few learners in step, and workgroups spread
evenly over the compute units.  Every element against the oracle, or against the two separate
calls."""
import pytest

import test_gpu_d1d_one_pass
import test_gpu_short_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
psgd = test_gpu_short_rows.psgd
mods = test_gpu_d1d_one_pass.mods


# learners times column groups: 24 000 per compute unit with the distance, 100 000 without (256 compute units)
@pytest.mark.parametrize("n,d,deg,gkind,extra", [
    (3, 8_191_996, 3, "f32", None), (3, 8_192_001, 3, "bf16", (1, 2, 3)), (4, 6_143_997, 3, "bf16", None), (4, 6_144_002, 3, "f32", None),
    (5, 4_915_201, 3, "f32", (3, 1, 2)), (6, 4_096_003, 3, "bf16", None), (6, 17_066_668, 3, "f32", None), (7, 3_510_859, 3, "f32", None),
    (8, 3_071_996, 3, "bf16", None), (8, 12_799_997, 3, "f32", (1, 2, 3)),
    (3, 8_192_004, -3, "f32", None), (4, 6_144_001, -3, "bf16", (1, 2, 3)), (5, 4_915_204, -3, "bf16", None), (7, 3_510_861, -3, "f32", None),
    (8, 12_800_004, -3, "f32", None),
    # the tiles of those by form: four rows per lane without the distance (the last place of seven learners has no row), two rows with it
    (6, 4_096_001, -3, "bf16", (1, 2, 3)), (6, 17_066_672, -3, "f32", None), (7, 14_628_576, -3, "f32", None), (7, 14_628_573, -3, "bf16", (1, 2, 3))])
def test_ring_walk_of_few_learners(psgd, n, d, deg, gkind, extra):
    test_gpu_short_rows.test_short_rows_every_element(psgd, n, d, deg, gkind, extra)


@pytest.mark.parametrize("n,d,deg,extra", [
    # a tile per workgroup: two, four, six and eight rows per lane; four, five and seven columns
    (2, 4, 3, 0), (3, 5, 3, 2), (7, 7, -3, 0), (16, 20_003, 3, 1), (4, 1_100_001, 3, 0), (5, 700_002, -3, 3), (6, 1_000_000, 3, 0),
    (8, 600_003, 3, 1), (12, 250_001, 3, 0), (64, 100_002, -3, 1), (300, 10_001, 3, 0),
    # large workgroups on narrow tiles, which leave it to the producer
    (512, 15_003, 3, 0),
    # looping: two, three and four rows per lane, whole tiles and a ragged last one, rows off the lines
    (8, 2_900_000, 3, 0), (7, 3_400_003, -3, 1), (13, 900_004, 3, 0), (33, 300_001, 3, 2), (64, 160_000, 3, 0), (64, 160_001, -3, 1), (128, 120_003, 3, 0),
    (300, 60_001, 3, 3), (512, 40_000, -3, 0),
    # off the lines on segments of 128 and 256 bytes: on either side of where the producer takes them
    (500, 26_999, 3, 0), (500, 27_001, -3, 1), (257, 52_529, -3, 0), (257, 52_531, 3, 2), (150, 50_001, 3, 1), (300, 30_002, -3, 3),
    # the ring walk from its line for this schedule on, rings and other tables
    (4, 6_144_001, 3, 0), (5, 4_915_205, 3, 1), (8, 3_072_004, 3, 0), (8, 3_072_001, -3, 0), (9, 1_536_001, 3, 0), (12, 1_228_804, -3, 0),
    # its other tables' tiles: of three rows up to 384 learners, of four with the next gradients in front of them beyond
    (384, 196_608, -3, 0), (385, 196_608, -3, 0), (385, 196_613, -3, 1), (512, 196_610, -3, 2), (450, 196_611, 3, 0),
    (16, 921_601, 3, 2), (32, 450_563, 3, 0), (64, 225_284, -3, 0), (128, 225_281, 3, 1), (128, 225_285, -3, 0)])
def test_next_gradients_beside_the_step(mods, n, d, deg, extra):
    test_gpu_d1d_one_pass.test_one_pass_is_the_two_calls(mods, n, d, deg, extra)


# global averaging in step from 12 000 column groups of all learners per compute unit on; workgroups spread evenly over the
# compute units (one, two and three on each) and left at 198, 293, 684 and 977 of 256 lanes; the distance of two and three learners on either side of 10 000 column groups per compute unit
@pytest.mark.parametrize("n,d,gkind,extra", [
    (3, 4_095_996, "f32", None), (3, 4_096_001, "bf16", (1, 2, 3)), (4, 3_072_003, "f32", None), (5, 2_457_602, "bf16", None),
    (6, 2_048_004, "f32", (3, 1, 2)), (7, 1_755_431, "f32", None), (8, 1_536_001, "bf16", None), (8, 1_535_996, "f32", None),
    (73, 202_100, "bf16", None), (33, 300_003, "f32", (1, 2, 3)), (16, 700_000, "f32", None), (9, 1_000_001, "bf16", None), (20, 524_289, "f32", None),
    (21, 538_821, "bf16", None), (77, 271_744, "f32", (1, 0, 3)), (120, 150_001, "bf16", None), (25, 420_003, "f32", None),
    (2, 10_239_996, "f32", None), (2, 10_240_001, "f32", None), (3, 10_240_004, "f32", None), (3, 10_260_003, "f32", (1, 0, 2))])
def test_global_average_and_distance(psgd, n, d, gkind, extra):
    test_gpu_short_rows.test_global_average_and_distance_with_rows_spread_over_lanes(psgd, n, d, gkind, extra)
