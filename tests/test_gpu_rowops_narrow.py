"""The row-wise kernels that give a wave a row (up to 2048 columns), at the edges of their vectors per
lane, of the rules that choose them and of their work-groups' row teams."""
import pytest

import test_gpu_rowops as base

pytestmark = pytest.mark.gpu

# columns: one lane; a ragged, full and just exceeded number of vectors per lane (512 columns each);
# the last width of a wave and the first of a work-group.  rows: one, an odd number over several
# teams, either side of 1024 (from which the backward of more than 1024 columns uses waves) and of
# 16384 (two backward work-groups per compute unit)
SHAPES = [(1, 8), (3, 384), (9, 512), (17, 520), (1030, 1024), (1023, 1032), (1025, 1032), (1024, 1536),
          (1031, 1544), (2050, 2048), (1029, 2056), (16385, 264), (16384, 504)]


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_narrow_rows(rows, cols):
    base.test_rmsnorm_fwd(rows, cols)
    base.test_layernorm_fwd_bwd(rows, cols)
