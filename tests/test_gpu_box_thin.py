"""GPU: the box passes on levels that cut a 16 x 8 x 4 box along x or y and
take boxes deeper along y or z instead, whole and cut off, and whose boxes are
counted along two axes: one cycle through fld_precondition against the
textbook cycle on the oracle's operator and against the marching tiles (the
bounds of the other boxes' test), and the residuals of solves on them (a solve
to 1e-8 is no sharper than 4e-6 against the oracle on these grids, the oracle's
own included, so the iterates themselves say less)."""
import pytest

import test_gpu_box as tb
import test_gpu_directions as td

pytestmark = pytest.mark.gpu

fld = tb.fld

SHAPES = [  # ([z][y][x], levels): finest box (x, y, z)
    ((64, 256, 8), 2),    # 8 x 16 x 4
    ((256, 66, 4), 1),    # 4 x 16 x 4, the last of y cut to 2
    ((1024, 4, 32), 2),   # 16 x 4 x 8
    ((1030, 4, 34), 1),   # 16 x 4 x 8, cut to 2 along x and 6 along z
    ((2048, 6, 6), 1),    # 6 x 6 x 8
    ((4096, 4, 8), 2),    # 8 x 4 x 16
]


@pytest.mark.parametrize("shape,levels", SHAPES)
@pytest.mark.parametrize("prec,tri", [(0, 0), (1, 0), (1, 1)])
def test_thin_box_cycle(fld, oracle_mod, monkeypatch, prec, tri, shape, levels):
    tb.test_box_cycle_is_the_textbook_cycle(fld, oracle_mod, monkeypatch, prec, tri, shape,
                                            levels)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [s for s, _ in SHAPES[:3]])
def test_thin_box_residuals(fld, shape, prec):
    """The residual that the box pass forms and sums: solves cut off after 1 ..
    6 iterations, the reported residual against b - A dE of the returned dE."""
    td.test_iterate_belongs_to_the_residual(fld, shape, 0, prec, 1)
