"""GPU: the lookup of a block's tile at the sizes where it changes its route: a
launch over at most 64 problems finds the block's problem by one load and a
ballot (64: every lane holds one), over more by a binary search.  Batches of
64, 65 and 100 tiny uneven problems, one step, bit for bit the steps of each
problem's own handle: a range taken wrongly does another problem's cells."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, log_case, params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fld():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1306_0645_amd as m
    return m


@pytest.mark.parametrize("n", [64, 65, 100])
@pytest.mark.parametrize("prec,nu", [(0, 1), (1, 1), (1, 2)])
def test_many_ranges(fld, n, prec, nu):
    log_case("ranges", n=n, prec=prec, nu=nu)
    rng = np.random.default_rng(81)
    shapes = [tuple(int(v) for v in rng.choice((4, 6, 8, 16), 3)) for _ in range(n)]
    ps = [synth.random_problem(s, 82 + i, sigma_ln=1.5, n_src=2, dt_factor=0.5)
          for i, s in enumerate(shapes)]
    prm = params(fld, ps[0], precision=prec, nu_pre=nu, nu_post=nu, cycle_switch=0)
    K, H = [dev(p["kappa"]) for p in ps], [dev(p["eta"]) for p in ps]
    Es = [dev(p["E"]) for p in ps]
    B = fld.Batch(shapes, [p["h"] for p in ps], prm)
    st = B.step(Es, K, H, [p["dt"] for p in ps])
    B.close()
    for i, p in enumerate(ps):
        S = fld.Solver(shapes[i], p["h"], prm)
        E = dev(p["E"])
        own = S.step(E, K[i], H[i], p["dt"])
        S.close()
        assert (st[i]["status"], st[i]["iters"]) == (0, own["iters"]), i
        assert np.array_equal(host(Es[i]), host(E)), (i, shapes[i])
