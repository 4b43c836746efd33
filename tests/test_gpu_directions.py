"""GPU: the fused PCG iteration stores its search direction, and updates the
iterate, every other time; a solve that stops after any number of iterations
has to return the iterate that its recursive residual belongs to.  Solves cut
off after 1 .. 6 iterations: ||b - A dE|| / ||b|| formed from the returned dE
against the reported recursive residual, which differ by rounding alone
(1e-12 of ||b||: a few iterations of FP64 recurrences; an update that was
lost, doubled or formed from the wrong direction is off by the residual's own
size, more than 1e-7 here)."""
import numpy as np
import pytest

import synth
from gpu_util import dev, log_case, params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fld():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1306_0645_amd as m
    return m


@pytest.mark.parametrize("shape,fused_tile_z", [((12, 20, 36), 0), ((24, 40, 96), 8),
                                                ((96, 194, 320), 4)])
@pytest.mark.parametrize("prec,d64", [(1, 1), (1, 0), (0, 1)])
def test_iterate_belongs_to_the_residual(fld, shape, fused_tile_z, prec, d64):
    """Boxes, marching tiles with the 64 x 4 SpMV tiles, and the fused-tile
    SpMV (2080 tiles)."""
    import torch
    log_case("directions", shape=shape, prec=prec, d64=d64)
    p = synth.random_problem(shape, 66, sigma_ln=1.5, n_src=3, dt_factor=2.0)
    E, K, H = dev(p["E"]), dev(p["kappa"]), dev(p["eta"])
    for m in range(1, 7):
        prm = params(fld, p, precision=prec, direction_fp64=d64, max_iter=m, rtol=1e-13,
                     cycle_switch=0, fused_tile_z=fused_tile_z, use_graph=m & 1)
        S = fld.Solver(shape, p["h"], prm)
        S.assemble(E, K, H, p["dt"])
        b = S.fld_get_system()["b"]
        dE, st = S.solve(check=False)
        assert st["status"] == fld.FLD_ENOCONV and st["iters"] == m
        r = float(torch.linalg.vector_norm(b - S.fld_apply(dE)) / torch.linalg.vector_norm(b))
        print(f"[directions] m={m} recursive={st['rel_resid']:.6e} formed={r:.6e}", flush=True)
        assert st["rel_resid"] > 1e-7 or m > 3
        assert abs(r - st["rel_resid"]) <= 1e-12
        S.close()
