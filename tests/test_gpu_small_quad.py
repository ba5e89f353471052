"""Small dense systems with M in registers (a quad of lanes per row): parity
with the FP64 oracle at the edges of its shapes, and independence of how the
steps are cut into launches."""
import numpy as np
import pytest

import fth_inputs as fi
import oracle
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


def normwise(a, b):
    den = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / den) if den > 0 else float(np.max(np.abs(a)))


def problem(n, gle):
    M, lam = fi.haar_spd(n, 50 + n, 0.1, 12.1) if n > 1 else (np.array([[2.5]]), np.array([2.5]))
    return M, fi.dt_rule(float(lam.max())), fi.white_noise_gle(1.0, 1.0) if gle == "white" else fi.load_gle(gle)


@pytest.mark.parametrize("n, R, prec, gle, quad", [
    (1, 1, fth.FTH_FP64, "white", True),
    (15, 4, fth.FTH_FP32, "invsqrt_ns4", True),
    (16, 2, fth.FTH_FP64, "invsqrt_ns4", True),
    (64, 64, fth.FTH_FP32, "invsqrt_ns4", True),
    (65, 1, fth.FTH_FP32, "invsqrt_ns4", True),
    (65, 8, fth.FTH_FP64, "ln_p_ns8", True),
    (128, 32, fth.FTH_FP64, "invsqrt_ns4", True),
    (128, 2, fth.FTH_FP32, "ln_p_ns10", True),
    (129, 1, fth.FTH_FP64, "invsqrt_ns4", False),
    (128, 4, fth.FTH_FP64, "ln_p_ns10", True),    # the most LDS a shape takes
])
def test_parity_and_launch_cuts(n, R, prec, gle, quad):
    M, h, g = problem(n, gle)
    pairs = fi.random_pairs(n, 9, 4) if n > 1 else np.zeros((1, 2), dtype=np.int32)
    opts = dict(pairs=pairs, replicas=R, precision=prec, seed=11, stream_id=2, burn_in=3, block_len=7, acc_diag=True,
                acc_pp=True, acc_trace=True)
    sol = fth.Solver(M, g.A_p, g.C_p, h, **opts).run(300)
    assert ("small_dense_kernel_quad" in sol.kernel_name) == quad, sol.kernel_name
    orc = oracle.OracleRun(M, g.A_p, g.C_p, h, R, np.concatenate([pairs, fi.diag_pairs(n)]), seed=11, stream=2,
                           burn_in=3, block_len=7).run(300)
    tol = 1e-10 if prec == fth.FTH_FP64 else 1e-4   # the repository's bounds for trajectories of each form
    q, p, s = sol.state()
    blk, s1, s2, nb, step = sol.accumulators()
    k = len(pairs) + n
    for name, a, b in (("q", q, orc.q), ("p", p, orc.p), ("s", s, orc.s), ("acc", (s1 + blk)[:k], orc.s1 + orc.blk)):
        if b.size:
            assert normwise(a, b) <= tol, (name, normwise(a, b))
    assert step == 300 and nb == 297 // 7
    # traces: sums over the diagonal estimates of q and p
    tot = s1 + blk
    for t, off in ((0, len(pairs)), (2, k + len(pairs))):
        assert abs(tot[2 * k + t] - tot[off: off + n].sum()) <= 1e-12 * abs(tot[2 * k + t])
    # other cuts of the same 300 steps (a launch holds at most 256) give the same bits
    cut = fth.Solver(M, g.A_p, g.C_p, h, **opts).run(1).run(254).run(2).run(43)
    for a, b in zip(sol.state() + sol.accumulators()[:3], cut.state() + cut.accumulators()[:3]):
        assert np.array_equal(a, b)
