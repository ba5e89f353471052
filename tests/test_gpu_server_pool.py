"""Device memory of finished requests goes to later ones: results do not
depend on what ran before, and the memory is given back with the server."""
import numpy as np
import pytest
import torch

import fth_inputs as fi
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


def drain(srv, ids):
    for _ in range(2000):
        if all(srv.poll(i)["state"] >= fth.FTH_REQ_DONE for i in ids):
            return
        srv.tick()
    raise AssertionError("requests did not finish")


@pytest.mark.parametrize("kind", ["sparse", "dense", "fp64"])
def test_reused_memory_changes_nothing(kind):
    g = fi.load_gle("invsqrt_ns4")

    def request(n, seed):
        M = fi.dense_ggt(n, 3) if kind == "dense" else fi.banded_spd_csr(n, 3)
        lam = fi.power_lambda_max(M.astype(np.float64)) if kind == "dense" else fi.gershgorin_max(M)
        prec = {"sparse": fth.FTH_FP32, "dense": fth.FTH_FP32_BF16X3, "fp64": fth.FTH_FP64}[kind]
        return dict(M=M, A_p=g.A_p, C_p=g.C_p, dt=fi.dt_rule(lam), pairs=fi.random_pairs(n, 20, 4),
                    replicas=64 if kind == "dense" else 32, precision=prec, seed=seed, stream_id=1, burn_in=5,
                    block_len=10, target=1e-9, max_steps=60)

    torch.cuda.synchronize()
    srv = fth.Server(steps_per_tick=20)
    first = srv.submit(**request(700, 9))
    drain(srv, [first])
    ref = srv.result(first)
    for n in (650, 900, 700, 699):  # other sizes in between, two at a time
        ids = [srv.submit(**request(n, 5)), srv.submit(**request(700, 9))]
        drain(srv, ids)
        out = srv.result(ids[1])
        assert np.array_equal(out[0], ref[0]) and np.array_equal(out[1], ref[1])
    held = torch.cuda.mem_get_info()[0]
    srv.close()
    assert torch.cuda.mem_get_info()[0] >= held
