"""Device memory of a server as the device reports it: kept between requests,
given back with the server."""
import pytest
import torch

import fth_inputs as fi
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu

MB = 1 << 20


def free_memory():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def serve(srv, n):
    g = fi.load_gle("invsqrt_ns4")
    M = fi.banded_spd_csr(n, 3)
    i = srv.submit(M=M, A_p=g.A_p, C_p=g.C_p, dt=fi.dt_rule(fi.gershgorin_max(M)), pairs=fi.random_pairs(n, 20, 4),
                   replicas=32, target=1e-9, max_steps=40)
    for _ in range(1000):
        if srv.poll(i)["state"] >= fth.FTH_REQ_DONE:
            break
        srv.tick()
    assert srv.poll(i)["state"] == fth.FTH_REQ_DONE
    return srv.poll(i)["footprint"]


def test_memory_is_kept_and_given_back():
    warm = fth.Server(steps_per_tick=20)   # code objects, queues and whatever else the runtime keeps
    serve(warm, 60000)
    warm.close()
    before = free_memory()
    srv = fth.Server(steps_per_tick=20)
    size = serve(srv, 60000)
    assert size > 64 * MB
    assert free_memory() <= before - size // 2          # idle blocks
    srv.close()
    # what the runtime itself may keep of a few dozen allocations (2 MB pages)
    assert free_memory() >= before - 16 * MB


def test_a_small_budget_bounds_what_is_kept():
    srv = fth.Server(steps_per_tick=20)
    size = serve(srv, 60000)
    srv.close()
    before = free_memory()
    srv = fth.Server(hbm_budget=size + size // 4, steps_per_tick=20)
    for n in (60000, 20000, 45000, 30000, 59000):
        serve(srv, n)
        assert before - free_memory() <= size + size // 4 + 64 * MB   # page rounding of some thirty blocks
    srv.close()
