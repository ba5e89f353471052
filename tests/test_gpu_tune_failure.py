"""An autotuner run that ends early, for want of device memory, leaves the
state, the step counter and the accumulators where they were."""
import numpy as np
import pytest
import torch

import fth_inputs as fi
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


class Rationed:
    """A device allocator that has memory for `left` more blocks (None: any number)."""

    def __init__(self):
        self.left, self.taken = None, 0

        def alloc(nbytes, _user):
            if self.left == 0:
                return None
            self.left = None if self.left is None else self.left - 1
            self.taken += 1
            ptr = int(torch.cuda.caching_allocator_alloc(int(nbytes)))
            torch.cuda.current_stream().synchronize()
            return ptr

        def release(ptr, _user):
            torch.cuda.caching_allocator_delete(int(ptr))

        self.hook = fth.fth_allocator(fth.ALLOC_FN(alloc), fth.RELEASE_FN(release), None)


@pytest.mark.parametrize("traces", [False, True])
def test_a_tuner_that_fails_changes_nothing(traces):
    torch.cuda.synchronize()
    g = fi.load_gle("invsqrt_ns4")
    failed = 0
    for left in range(0, 60):
        M = fi.banded_spd_csr(1237 + left, 3)   # a size of its own: the tuner remembers its choices by size
        kw = dict(pairs=fi.random_pairs(M.n, 30, 1), replicas=8, seed=3, acc_diag=True, acc_trace=traces, block_len=6)
        h = fi.dt_rule(fi.gershgorin_max(M))
        ref = fth.Solver(M, g.A_p, g.C_p, h, **kw).run(12).run(13)
        mem = Rationed()
        sol = fth.Solver(M, g.A_p, g.C_p, h, allocator=mem.hook, tune=True, **kw)
        mem.left = left
        try:
            sol.run(12)
        except fth.FthError as e:
            assert e.status == fth.FTH_ENOMEM
            failed += 1
            mem.left = None
            sol.run(12)
        done = mem.left is not None
        sol.run(13)
        for a, b in zip(sol.state(), ref.state()):
            assert np.array_equal(a, b), left
        for a, b in zip(sol.accumulators()[:3], ref.accumulators()[:3]):
            # a tuned shape may add the FP64 products of a row in another order
            assert np.max(np.abs(a - b)) <= 2 * (8 * M.n + 25) * 2.0 ** -53 * np.max(np.abs(b)), left
        sol.close()
        if done:
            break
    assert done and failed >= 8
