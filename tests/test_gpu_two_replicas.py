"""Sparse step with two replicas per thread (an autotuner candidate): the two
lanes of a group of four replicas share its noise blocks.  Whatever shape the
tuner takes, the trajectory is the untuned one's bit for bit, and the
accumulators differ by the order of their FP64 sums only."""
import numpy as np
import pytest

import fth_inputs as fi
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu


def random_gle(ns, seed):
    rng = np.random.default_rng(seed)
    d = ns + 1
    K = rng.normal(size=(d, d))
    return (K - K.T) + np.diag(rng.uniform(0.3, 2.0, d)), 0.9 * np.eye(d)


@pytest.mark.parametrize("matrix", ["laplacian", "m1"])
@pytest.mark.parametrize("R, ns, prec", [(4, 4, fth.FTH_FP64), (4, 3, fth.FTH_FP32), (16, 8, fth.FTH_FP32),
                                         (32, 3, fth.FTH_FP64), (128, 0, fth.FTH_FP64)])
def test_tuned_trajectory_is_the_untuned_one(matrix, R, ns, prec):
    M = fi.laplacian3d_csr(9, 0.1) if matrix == "laplacian" else fi.m1_lattice_csr(7, 3, dtype=np.float32)
    h = fi.dt_rule(fi.gershgorin_max(M))
    A, C = random_gle(ns, 5)
    kw = dict(pairs=fi.random_pairs(M.n, 30, 1), replicas=R, seed=3, acc_diag=True, acc_pp=True, block_len=6,
              precision=prec)
    a = fth.Solver(M, A, C, h, tune=True, **kw).run(25)
    b = fth.Solver(M, A, C, h, tune=False, **kw).run(25)
    print(f"[two replicas] {a.kernel_name}", flush=True)
    for x, y in zip(a.state(), b.state()):
        assert np.array_equal(x, y)
    for x, y in zip(a.accumulators()[:3], b.accumulators()[:3]):
        # a sum of R products of FP64 terms in another order: R roundings of the absolute sum at most
        assert np.max(np.abs(x - y)) <= 2 * R * 2.0 ** -53 * 25 * np.max(np.abs(y))
