"""GPU: the V-cycle's tail (the levels that one workgroup sweeps, and the
coarsest solve) at the sizes where it changes its route: a coarsest level of
at most 64 cells (one wave), up to 1024 and 2048 (operator in registers),
4096, 8192 and 16384 (operator streamed) and beyond (vectors in memory), and
no, one, two or more smoothing levels above it, in LDS (one cell a thread, the
largest in pairs of cells) or in memory.  One
cycle through fld_precondition against the textbook cycle on the oracle's
operator, within the bounds of the cycle tests (the coarsest solve there:
sparse CG to 1e-14)."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla

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


def _solve(op, f):
    n = f.size
    A = spla.LinearOperator((n, n), matvec=lambda u: tv._apply(op, u.reshape(f.shape)).ravel(),
                            dtype=np.float64)
    M = spla.LinearOperator((n, n), matvec=lambda u: u / op[0].ravel(), dtype=np.float64)
    x, info = spla.cg(A, f.ravel(), rtol=1e-14, atol=0.0, maxiter=2000, M=M)
    assert info == 0
    return x.reshape(f.shape)


CASES = [  # (shape, levels, tail_cells): coarsest cells, smoothing levels of the tail
    ((8, 8, 8), 2, 512),       # 64, none: one wave
    ((8, 8, 12), 2, 512),      # 96, none
    ((16, 16, 24), 2, 512),    # 768, none
    ((20, 24, 24), 2, 512),    # 1440: two cells a thread
    ((28, 32, 32), 2, 512),    # 3584: four
    ((36, 40, 40), 2, 512),    # 7200: eight
    ((50, 50, 50), 2, 512),    # 15625, odd extents: sixteen
    ((56, 52, 56), 2, 512),    # 20384: in memory
    ((16, 16, 16), 3, 512),    # 64 under one level of 512 in LDS
    ((16, 16, 20), 3, 700),    # 80 under one of 640
    ((32, 16, 16), 4, 1024),   # 16 under levels of 1024 and 128 in LDS
    ((16, 16, 32), 4, 2048),   # 16 under 128 and 1024
    ((32, 32, 32), 4, 8192),   # 64 under levels of 4096 (in pairs) and 512 in LDS
    ((32, 32, 32), 3, 512),    # 512 right under one of 4096
    ((24, 20, 32), 3, 512),    # 240 under one of 1920, rows of 6 pairs
    ((24, 24, 48), 3, 512),    # 432 under one of 3456
    ((32, 32, 32), 5, 512),    # 8 under levels of 4096, 512 and 64
    ((32, 32, 64), 4, 8192),   # 128 under levels of 8192 and 1024 in memory
]


@pytest.mark.parametrize("shape,levels,tail_cells", CASES)
@pytest.mark.parametrize("nu", [1, 2])
@pytest.mark.parametrize("prec", [0, 1])
def test_tail_is_the_textbook_cycle(fld, oracle_mod, monkeypatch, prec, nu, shape, levels,
                                    tail_cells):
    log_case("tail", prec=prec, nu=nu, shape=shape, levels=levels, tail=tail_cells)
    monkeypatch.setattr(tv, "_solve_exact", _solve)
    p = synth.random_problem(shape, 63, sigma_ln=1.5, n_src=3, dt_factor=0.5)
    prm = params(fld, p, precision=prec, mg_levels=levels, nu_pre=nu, nu_post=nu,
                 cycle_switch=0, tail_cells=tail_cells, local_sweeps=0,
                 prolongation=1 if nu == 2 else 0)
    S = fld.Solver(p["shape"], p["h"], prm)
    S.assemble(dev(p["E"]), dev(p["kappa"]), dev(p["eta"]), p["dt"], p["a"], 0.0)
    f = np.random.default_rng(9).normal(size=shape)
    z = host(S.fld_precondition(dev(f)))
    D, Ax, Ay, Az, _ = oracle_problem(oracle_mod, p, prm).system()
    ops = [(D, (Ax, Ay, Az))]
    for _ in range(levels - 1):
        ops.append(tv._coarsen(ops[-1], prm.coarse_scale))
    zr = tv._vcycle(ops, 0, f, nu, trilinear=bool(prec) and nu == 2)
    err = rel_l2(z, zr)
    print(f"[tail] prec={prec} nu={nu} shape={shape} err={err:.2e}", flush=True)
    assert err <= (1e-9 if prec == 0 else 2e-5)
