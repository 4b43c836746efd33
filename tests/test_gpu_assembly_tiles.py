"""GPU: the assembly's tiles take the limiters of their -x and -y edges eight
planes at a time and list the local sweeps' cells on the way.  Grids whose
tiles are cut off in every direction (rows shorter than a wave, a few cells
beyond one, rows that do not fill a block) and tiles of 1 to 20 planes, so
that the last group of planes holds 1 to 8: the system against the oracle's
(both FP64, the same formulas: a few roundings, 1e-13), and the mixed cycle
with local sweeps against the textbook cycle, within the bound of the cycle
tests."""
import numpy as np
import pytest

import synth
import test_gpu_vcycle as tv
from gpu_util import dev, host, log_case, oracle_problem, params, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fld():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1306_0645_amd as m
    return m


@pytest.mark.parametrize("shape,tile_z", [((6, 10, 34), 0), ((20, 10, 130), 20), ((18, 6, 66), 9),
                                          ((10, 14, 62), 1), ((24, 6, 4), 16)])
@pytest.mark.parametrize("prec", [0, 1])
def test_system_matches_oracle(fld, oracle_mod, shape, tile_z, prec):
    log_case("assembly_tiles", shape=shape, tile_z=tile_z, prec=prec)
    p = synth.random_problem(shape, 17, sigma_ln=1.5, n_src=3, dt_factor=0.05)
    dx = p["h"][0]
    p["h"] = (dx, 1.25 * dx, 0.8 * dx)
    prm = params(fld, p, precision=prec, tile_z=tile_z)
    S = fld.Solver(shape, p["h"], prm)
    S.assemble(dev(p["E"]), dev(p["kappa"]), dev(p["eta"]), p["dt"], p["a"], p["adot"])
    got = {k: host(v) for k, v in S.fld_get_system().items()}
    diag, Ax, Ay, Az, b = oracle_problem(oracle_mod, p, prm).system()
    np.testing.assert_allclose(got["diag"], diag, rtol=1e-13)
    for g, w in ((got["Tx"], Ax), (got["Ty"], Ay), (got["Tz"], Az)):
        np.testing.assert_allclose(g, w, rtol=1e-13, atol=1e-16 * np.abs(w).max())
    np.testing.assert_allclose(got["b"], b, rtol=0, atol=1e-12 * np.abs(b).max())


@pytest.mark.parametrize("shape,tile_z", [((24, 12, 70), 20), ((22, 10, 34), 9), ((16, 18, 66), 0)])
def test_listed_cells_are_the_coupled_ones(fld, oracle_mod, shape, tile_z):
    log_case("assembly_lists", shape=shape, tile_z=tile_z)
    p = synth.random_problem(shape, 62, sigma_ln=1.5, n_src=3, dt_factor=2.0)
    prm = params(fld, p, precision=1, mg_levels=2, nu_pre=1, nu_post=1, cycle_switch=0,
                 tile_z=tile_z, prolongation=0, local_sweeps=1, local_coupling=0.9)
    S = fld.Solver(shape, p["h"], prm)
    S.assemble(dev(p["E"]), dev(p["kappa"]), dev(p["eta"]), p["dt"], p["a"], 0.0)
    f = np.random.default_rng(8).normal(size=shape)
    z = host(S.fld_precondition(dev(f)))
    D, Ax, Ay, Az, _ = oracle_problem(oracle_mod, p, prm).system()
    ops = [(D, (Ax, Ay, Az))]
    ops.append(tv._coarsen(ops[0], prm.coarse_scale))
    err = rel_l2(z, tv._vcycle(ops, 0, f, 1, local=(1, 0.9)))
    off = rel_l2(z, tv._vcycle(ops, 0, f, 1, local=(0, 0.9)))
    frac = tv._local_mask(ops[0], 0.9).mean()
    print(f"[assembly lists] listed={frac:.3f} err={err:.2e} without={off:.2e}", flush=True)
    assert err <= 2e-5
    assert frac > 0.002 and off > 10 * err
