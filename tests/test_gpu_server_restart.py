"""GPU: a served solve that restarts from its true residual in the tick in
which another request ends, whose tables are rebuilt before the next one: the
restarted solve still owes its finest down pass.  Optically thin boxes over
long steps (they restart, and each ends in a tick of its own), admitted
together, bit for bit against each one served alone."""
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


@pytest.mark.parametrize("d64", [1, 0])
def test_restart_survives_a_rebuild(fld, d64):
    import torch
    log_case("server_restart", d64=d64)
    ps = [synth.thin_uniform_problem(16, 5e6, seed=s) for s in range(32)]
    prm = params(fld, ps[0], precision=1, direction_fp64=d64, rtol=3e-9, max_iter=400,
                 max_dt_cuts=0, cycle_switch=0, warm_start=0)
    dp = [(dev(p["E"]), dev(p["kappa"]), dev(p["eta"])) for p in ps]
    torch.cuda.synchronize()
    srv = fld.Server(prm, 1 << 30)

    def serve(i):
        out = torch.zeros_like(dp[i][0])
        return out, srv.submit(ps[i]["shape"], ps[i]["h"], *dp[i], out, ps[i]["dt"])

    alone, iters = [], []
    for i in range(len(ps)):
        out, t = serve(i)
        srv.drain()
        res = srv.poll(t)
        alone.append(host(out))
        iters.append((res["status"], res["iters"]))
    print(f"[server restart] (status, iters)={iters}", flush=True)
    assert len(set(iters)) > 8  # (requests end in different ticks)
    mixed = [serve(i) for i in range(len(ps))]
    srv.drain()
    got = [srv.poll(t) for _, t in mixed]
    srv.close()
    for i, (out, _) in enumerate(mixed):
        assert (got[i]["status"], got[i]["iters"]) == iters[i], i
        assert np.array_equal(host(out), alone[i]), i
