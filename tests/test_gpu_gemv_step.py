"""Dense steps of few replicas in one launch (matrix-vector products and the
row update together): parity with the FP64 oracle where rows and columns do
not fill a workgroup's share, with every estimator, and independence of how
the steps are cut into chunks."""
import numpy as np
import pytest

import fth_inputs as fi
import oracle
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


def normwise(a, b):
    den = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / den) if den > 0 else float(np.max(np.abs(a)))


@pytest.mark.parametrize("n, R, prec", [(4097, 1, fth.FTH_FP32), (2051, 2, fth.FTH_FP64), (1025, 4, fth.FTH_FP64),
                                        (1030, 4, fth.FTH_FP32), (513, 8, fth.FTH_FP32), (514, 8, fth.FTH_FP64)])
def test_one_launch_step(n, R, prec):
    M = fi.dense_ggt(n, 7 + n)
    M64 = M.astype(np.float64)
    h = fi.dt_rule(fi.power_lambda_max(M64))
    g = fi.load_gle("ln_p_ns8" if n < 1000 else "invsqrt_ns4")
    pairs = fi.random_pairs(n, 300, 8)
    opts = dict(pairs=pairs, replicas=R, precision=prec, seed=3, stream_id=2, burn_in=2, block_len=4, acc_diag=True,
                acc_pp=True, acc_trace=True)
    sol = fth.Solver(M, g.A_p, g.C_p, h, steps_per_graph=6, **opts).run(21)
    assert sol.kernel_name.startswith("dense_gemv_kernel"), sol.kernel_name
    orc = oracle.OracleRun(M64, g.A_p, g.C_p, h, R, np.concatenate([pairs, fi.diag_pairs(n)]), seed=3, stream=2,
                           burn_in=2, block_len=4).run(21)
    tol = 1e-10 if prec == fth.FTH_FP64 else 1e-4   # the repository's bounds for trajectories of each form
    q, p, s = sol.state()
    blk, s1, s2, nb, step = sol.accumulators()
    k = len(pairs) + n
    tot = s1 + blk
    for name, a, b in (("q", q, orc.q), ("p", p, orc.p), ("s", s, orc.s), ("acc", tot[:k], orc.s1 + orc.blk)):
        assert normwise(a, b) <= tol, (name, normwise(a, b))
    for t, off in ((0, len(pairs)), (2, k + len(pairs))):  # traces: sums of the diagonal estimates of q and p
        assert abs(tot[2 * k + t] - tot[off: off + n].sum()) <= 1e-12 * abs(tot[2 * k + t])
    # chunks of other lengths (the rows are taken forward on even steps, backward on odd ones)
    cut = fth.Solver(M, g.A_p, g.C_p, h, steps_per_graph=3, **opts).run(5).run(1).run(15)
    for a, b in zip(sol.state(), cut.state()):
        assert np.array_equal(a, b)
    for a, b in zip(sol.accumulators()[:3], cut.accumulators()[:3]):
        assert np.array_equal(a, b)
