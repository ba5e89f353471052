"""A dense matrix is laid out on the device, in parts of rows when it is large:
the same bits from FP32 and FP64 sources, in one part and in several."""
import numpy as np
import pytest

import fth_inputs as fi
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [fth.FTH_FP64, fth.FTH_FP32_BF16X3], ids=["fp64", "bf16x3"])
@pytest.mark.parametrize("n, R", [(1031, 32), (2901, 16), (2901, 2), (130, 64)])
def test_layout_from_either_source(n, R, prec):
    """2901 rows are two parts of 64 MB as doubles (the copy that a context
    without a replica count keeps) and one as floats."""
    M = fi.dense_ggt(n, 5)
    h = fi.dt_rule(fi.power_lambda_max(M.astype(np.float64)))
    g = fi.load_gle("invsqrt_ns4")
    kw = dict(precision=prec, seed=3, acc_diag=True, block_len=2)
    a = fth.Solver(M, g.A_p, g.C_p, h, replicas=R, **kw).run(4)
    b = fth.Solver(M, g.A_p, g.C_p, h, **kw).run(4, replicas=R)
    q = np.random.default_rng(1).normal(size=(n, R)).astype(np.float32).astype(np.float64)
    fa, fb = a.force(q), b.force(q)
    assert np.array_equal(fa, fb)
    ref = -(M.astype(np.float64) @ q)
    # the bounds of the two force forms against an FP64 product
    assert np.max(np.abs(fa - ref)) <= (1e-13 if prec == fth.FTH_FP64 else 3e-5) * np.max(np.abs(ref))
    for x, y in zip(a.state() + a.accumulators()[:3], b.state() + b.accumulators()[:3]):
        assert np.array_equal(x, y)
