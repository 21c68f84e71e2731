"""The tiled kernel: tables of other than three slots on long rows, for the numbers of learners that take it, none of which fills its tiles
exactly: places without a row in the last row group, rows that the lanes of a column take unevenly, row segments of 512 bytes to 4 KB, rows on lines and (29 to 32 learners, or
longer rows from 16 slots on) off them, with columns left over.  Every element and the distance against the oracle's sparse form, out of place and in
place.  Which tables take it: the check of the launch arithmetic."""
import pytest

import test_gpu_short_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
psgd = test_gpu_short_rows.psgd


@pytest.mark.parametrize("n,d,deg,gkind,extra", [
    # on lines; 13 to 16 learners with the distance only
    (13, 1_572_896, 20, "bf16", None), (14, 1_600_032, 16, "f32", None), (15, 1_572_864, 32, "f32", (32, 0, 5)),
    # 23 to 28 and 43 to 48 learners without it
    (23, 1_572_864, 16, "f32", None), (25, 1_572_864, 14, "bf16", None), (27, 1_580_064, 23, "f32", None), (43, 1_572_896, 18, "f32", None), (47, 1_572_896, 23, "bf16", None),
    # off lines, whole and ragged column groups
    (29, 1_572_865, 13, "f32", (1, 2, 3)), (30, 1_600_003, 5, "bf16", None), (31, 1_600_004, 4, "f32", None), (32, 1_572_866, 9, "bf16", (3, 0, 1)),
    (49, 1_572_896, 4, "f32", None), (53, 1_572_896, 5, "bf16", None), (63, 1_572_864, 13, "f32", None),
    (65, 1_572_896, 16, "bf16", None), (100, 1_572_896, 17, "f32", None), (113, 1_572_896, 5, "f32", None), (127, 1_572_864, 9, "bf16", None),
    # longer rows that start on 16 bytes only
    (14, 3_145_732, 16, "f32", None), (26, 3_145_732, 24, "bf16", None), (50, 3_145_740, 20, "bf16", None)])
def test_tiled_rows_every_element(psgd, n, d, deg, gkind, extra):
    on_lines = extra is not None and extra[0] % 32 == 0           # pitched rows that stay on lines
    test_gpu_short_rows.every_element(psgd, n, d, deg, gkind, extra, 32 if on_lines else 1 if extra else 0)
