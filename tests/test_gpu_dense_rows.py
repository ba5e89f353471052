"""Dense steps on the matrix cores in one launch (16 rows and a group of
columns per workgroup): parity with the FP64 oracle where rows, columns and
k-steps do not fill a workgroup's share, on both sides of the dispatch's
line, with every estimator, and independence of the chunking."""
import numpy as np
import pytest

import fth_inputs as fi
import oracle
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu

SPLIT, F64 = fth.FTH_FP32_BF16X3, fth.FTH_FP64


def normwise(a, b):
    den = np.max(np.abs(b))
    return float(np.max(np.abs(a - b)) / den) if den > 0 else float(np.max(np.abs(a)))


@pytest.mark.parametrize("n, R, prec, gle, name", [
    (257, 16, SPLIT, "invsqrt_ns4", "dense_rows_bf16x3_kernel<NS=4,CT=1>"),
    (641, 32, SPLIT, "ln_p_ns10", "dense_rows_bf16x3_kernel<NS=10,CT=1>"),
    (520, 128, SPLIT, "invsqrt_ns4", "dense_rows_bf16x3_kernel<NS=4,CT=2>"),
    (1571, 128, SPLIT, "invsqrt_ns4", "dense_rows_bf16x3_kernel<NS=4,CT=4>"),   # n^2 R just below 3.2e8
    (1585, 128, SPLIT, "invsqrt_ns4", "gemm_bf16x3_kernel"),                     # and just above
    (271, 16, F64, "ln_p_ns10", "dense_rows_f64_kernel<NS=10,CT=1>"),
    (560, 128, F64, "invsqrt_ns4", "dense_rows_f64_kernel<NS=4,CT=2>"),
    (1249, 64, F64, "invsqrt_ns4", "dense_rows_f64_kernel<NS=4,CT=2>"),          # just below 1e8
    (1260, 64, F64, "invsqrt_ns4", "gemm_f64_kernel"),
])
def test_one_launch_step(n, R, prec, gle, name):
    M = fi.dense_ggt(n, 3 + n)
    M64 = M.astype(np.float64)
    h = fi.dt_rule(fi.power_lambda_max(M64))
    g = fi.load_gle(gle)
    pairs = fi.random_pairs(n, 45, 8)
    opts = dict(pairs=pairs, replicas=R, precision=prec, seed=3, stream_id=2, burn_in=2, block_len=4, acc_diag=True,
                acc_pp=True, acc_trace=True)
    sol = fth.Solver(M, g.A_p, g.C_p, h, steps_per_graph=6, **opts).run(21)
    assert sol.kernel_name.startswith(name), sol.kernel_name
    orc = oracle.OracleRun(M64, g.A_p, g.C_p, h, R, np.concatenate([pairs, fi.diag_pairs(n)]), seed=3, stream=2,
                           burn_in=2, block_len=4).run(21)
    tol = 1e-10 if prec == F64 else 1e-4   # the repository's bounds for trajectories of each form
    q, p, s = sol.state()
    blk, s1, s2, nb, step = sol.accumulators()
    k = len(pairs) + n
    tot = s1 + blk
    for what, a, b in (("q", q, orc.q), ("p", p, orc.p), ("s", s, orc.s), ("acc", tot[:k], orc.s1 + orc.blk)):
        assert normwise(a, b) <= tol, (what, normwise(a, b))
    for t, off in ((0, len(pairs)), (2, k + len(pairs))):  # traces: sums of the diagonal estimates of q and p
        assert abs(tot[2 * k + t] - tot[off: off + n].sum()) <= 1e-12 * abs(tot[2 * k + t])
    # other chunks, and a continuation from an image saved at an odd step, give the same bits
    cut = fth.Solver(M, g.A_p, g.C_p, h, steps_per_graph=3, **opts).run(5).run(2)
    rest = fth.Solver(M, g.A_p, g.C_p, h, **opts)
    rest.load(cut.save())
    for other in (cut.run(14), rest.run(14)):
        for a, b in zip(sol.state(), other.state()):
            assert np.array_equal(a, b)
        for a, b in zip(sol.accumulators()[:3], other.accumulators()[:3]):
            assert np.array_equal(a, b)
