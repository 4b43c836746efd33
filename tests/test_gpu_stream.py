"""GPU: streaming access, which the launches take when the problems of a handle
or a batch together need more than 400 MB: three problems below that size, each
in its own handle (cached) and all in one batch (streaming), two steps, bit for
bit the same; on boxes and on marching tiles, warm-started, in every storage
form and with the cycles whose update of x is a pass of its own."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, log_case, params

pytestmark = pytest.mark.gpu

SHAPES = [(112, 96, 128), (120, 116, 120), (128, 108, 120)]


@pytest.fixture(scope="module")
def fld():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1306_0645_amd as m
    return m


@pytest.fixture(scope="module")
def problems():
    return [synth.random_problem(s, 91 + i, sigma_ln=1.5, n_src=3, dt_factor=0.5)
            for i, s in enumerate(SHAPES)]


@pytest.mark.parametrize("kw", [
    {"precision": 0}, {"precision": 0, "nu_pre": 2, "nu_post": 2, "warm_start": 1},
    {"precision": 1, "prolongation": 1}, {"precision": 1, "direction_fp64": 0},
    {"precision": 1, "nu_pre": 2, "nu_post": 2},
    {"precision": 1, "direction_fp64": 0, "nu_pre": 2, "nu_post": 2}])
def test_streaming_changes_nothing(fld, problems, kw):
    log_case("stream", **kw)
    ps = problems
    prm = params(fld, ps[0], cycle_switch=0, **kw)
    sizes = [fld.fld_workspace_bytes(fld.make_grid(s, p["h"]), prm)
             for s, p in zip(SHAPES, ps)]
    assert max(sizes) < 400 << 20 < sum(sizes) - (1 << 20)
    K, H = [dev(p["kappa"]) for p in ps], [dev(p["eta"]) for p in ps]
    Es = [dev(p["E"]) for p in ps]
    B = fld.Batch(SHAPES, [p["h"] for p in ps], prm)
    st = [B.step(Es, K, H, [p["dt"] for p in ps]) for _ in range(2)]
    B.close()
    for i, p in enumerate(ps):
        S = fld.Solver(SHAPES[i], p["h"], prm)
        E = dev(p["E"])
        for s in st:
            own = S.step(E, K[i], H[i], p["dt"])
            assert (s[i]["status"], s[i]["iters"]) == (0, own["iters"]), i
        S.close()
        assert np.array_equal(host(Es[i]), host(E)), i
