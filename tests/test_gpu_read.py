"""Readout formed on the device: equal, bit for bit, to the block-average
formulas evaluated on the host from the raw accumulators (the same FP64
operations in the same order), at the edges of the readout chunks."""
import numpy as np
import pytest

import fth_inputs as fi
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


def host_read(sol, R, L, burn_in):
    blk, s1, s2, nb, step = sol.accumulators()
    nacc = max(0, step - burn_in)
    with np.errstate(invalid="ignore", divide="ignore"):
        est = (s1 + blk) / (R * float(nacc)) if nacc else np.full_like(s1, np.nan)
        if nb < 2:
            return est, np.full_like(s1, np.inf), nacc
        sc = 1.0 / (R * float(L))
        sb, sbb = s1 * sc, s2 * sc * sc
        var = (sbb - sb * sb / float(nb)) / float(nb - 1)
        return est, np.sqrt(np.where(var < 0.0, 0.0, var) / float(nb)), nacc


@pytest.mark.parametrize("n, npairs, diag", [(4, 1, False), (32767, 0, True), (32760, 8, True), (32769, 0, True),
                                             (65530, 7, True)])
@pytest.mark.parametrize("steps", [0, 7, 23])
def test_read_equals_host_formula(n, npairs, diag, steps):
    M = fi.banded_spd_csr(n, 5)
    g = fi.load_gle("invsqrt_ns4")
    pairs = fi.random_pairs(n, npairs, 6) if npairs else None
    sol = fth.Solver(M, g.A_p, g.C_p, 0.02, pairs=pairs, replicas=4, seed=3, burn_in=2, block_len=5, acc_diag=diag)
    sol.run(0)
    if steps:
        sol.run(steps)
    est, se, nacc = sol.read()
    ref, ref_se, ref_n = host_read(sol, 4, 5, 2)
    assert len(est) == npairs + (n if diag else 0) and nacc == ref_n
    assert np.array_equal(est, ref, equal_nan=True) and np.array_equal(se, ref_se)
    again = sol.read()
    assert np.array_equal(again[0], est, equal_nan=True) and np.array_equal(again[1], se)
    sol.close()
