"""GPU: solves cut off after 1 .. 6 iterations on the fused-tile SpMV, which a
grid takes from 2048 fused tiles on (2 x 13 x 80 here, the extents of 96 and
194 cut the tiles; the host check of the routes pins it): the skipped and the
stored direction, and the iterate's pending updates, in both direction
precisions, as for the other SpMV tilings (the same bound)."""
import pytest

import test_gpu_directions as td

pytestmark = pytest.mark.gpu

fld = td.fld


@pytest.mark.parametrize("d64", [1, 0])
def test_iterate_belongs_to_the_residual(fld, d64):
    td.test_iterate_belongs_to_the_residual(fld, (320, 194, 96), 4, 1, d64)
