"""Workspace sizes on the host (no GPU): no grid needs more than the sizes
below, which an earlier layout of the tables took, so that a grid that fitted
a workspace of the caller's, a server's arena or the 64 MiB of
fld_step_static still fits; among them grids just under that line.  Every
box of the box passes fits the buffers that the kernels hold it in, and every
level takes the route that the rules give it."""
import pytest

from test_carve_host import _run_host


@pytest.fixture(scope="module")
def fld():
    import paper_1306_0645_amd as m
    return m


SIZES = [  # (shape [z][y][x], parameters, bytes)
    ((2756, 42, 4), {}, 67071744),
    ((6, 186, 384), {"precision": 1, "nu_pre": 2, "nu_post": 2}, 70529536),
    ((6, 178, 364), {"precision": 1}, 67107328),
    ((4, 4, 4), {}, 15616),
    ((8, 8, 8), {"precision": 1}, 84736),
    ((32, 32, 32), {}, 3921920),
    ((32, 32, 32), {"precision": 1}, 4877824),
    ((64, 64, 64), {"precision": 1}, 38956288),
    ((32, 32, 32), {"tile_z": 64, "nu_pre": 2, "nu_post": 2}, 3906560),
    ((64, 64, 64), {"precision": 1, "smoother": 1}, 38057472),
    ((96, 64, 40), {}, 29384192),
    ((200, 200, 200), {"precision": 1, "direction_fp64": 0}, 1121217792),
    ((128, 128, 128), {"precision": 1, "fused_levels": 1}, 310749440),
    ((256, 256, 256), {}, 1995265792),
    ((640, 640, 640), {"precision": 1, "mg_levels": 6}, 38815165440),
    ((3420, 92, 4), {"nu_pre": 2, "nu_post": 2}, 181725440),
    ((9422, 4, 40), {"precision": 1}, 259671808),
    ((4, 1050, 234), {}, 141846272),
    ((212, 212, 212), {"precision": 1, "tile_z": 64, "fused_tile_z": 256}, 1413878016),
    ((512, 4, 4), {"precision": 1, "mg_levels": 2}, 1348608),
    ((20, 36, 500), {"tail_cells": 0}, 43147008),
]


@pytest.mark.parametrize("shape,kw,size", SIZES)
def test_no_grid_needs_more(fld, shape, kw, size):
    p = fld.fld_default_params(3e10, 1.0, **kw)
    assert 0 < fld.fld_workspace_bytes(fld.make_grid(shape, (1.0, 1.0, 1.0)), p) <= size


def test_boxes_fit_their_buffers(tmp_path):
    _run_host(tmp_path, "box_shapes")


def test_level_routes(tmp_path):
    _run_host(tmp_path, "level_routes")
