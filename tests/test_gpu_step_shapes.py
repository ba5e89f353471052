"""Sparse one-step kernels at two replicas per thread, where the two lanes of a
group of four replicas share its noise blocks: each form (coded, plain, long
rows) at odd and even numbers of extra momenta, with the shape fixed instead of
left to the autotuner.  Parity with the FP64 oracle, and bit for bit the
trajectory of the default shape."""
import ctypes

import numpy as np
import pytest

import fth_inputs as fi
import oracle
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu

TOL = {fth.FTH_FP64: 1e-10, fth.FTH_FP32: 1e-4}   # the repository's bounds for trajectories


def random_gle(ns, seed):
    rng = np.random.default_rng(seed)
    d = ns + 1
    K = rng.normal(size=(d, d))
    return (K - K.T) + np.diag(rng.uniform(0.3, 2.0, d)), 0.9 * np.eye(d)


def fix_shape(sol, threads, per_thread, streaming):
    f = fth.lib().fth_internal_step_shape
    f.restype, f.argtypes = ctypes.c_int32, [ctypes.c_void_p] + [ctypes.c_int32] * 3
    fth._check(f(sol.ctx, threads, per_thread, streaming))
    return sol


@pytest.mark.parametrize("form", ["coded", "plain", "long"])
@pytest.mark.parametrize("prec", [fth.FTH_FP32, fth.FTH_FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("R, ns, threads, streaming", [(4, 0, 64, 0), (4, 3, 256, 0), (8, 4, 128, 1), (32, 7, 64, 0),
                                                       (128, 1, 256, 1), (16, 10, 128, 0)])
def test_two_replicas_per_thread(form, prec, R, ns, threads, streaming):
    M = fi.m1_lattice_csr(6, 3, dtype=np.float64) if form == "long" else fi.laplacian3d_csr(7, 0.1, dtype=np.float64)
    h = fi.dt_rule(fi.gershgorin_max(M))
    A, C = random_gle(ns, 5)
    pairs = fi.random_pairs(M.n, 30, 1)
    kw = dict(pairs=pairs, replicas=R, seed=3, acc_diag=True, acc_pp=True, acc_trace=True, burn_in=2, block_len=6,
              precision=prec, coded_matrix=0 if form == "coded" else -1)
    sol = fix_shape(fth.Solver(M, A, C, h, steps_per_graph=8, **kw), threads, 2, streaming).run(25)
    name = sol.kernel_name
    assert f"RPT=2,NT={streaming},CODED={int(form == 'coded')}> block={threads}" in name, name
    assert ("(long-row batches)" in name) == (form == "long"), name
    ref = fth.Solver(M, A, C, h, **kw).run(25)
    assert "RPT=4" in ref.kernel_name
    for a, b in zip(sol.state(), ref.state()):
        assert np.array_equal(a, b)
    tot = [x.accumulators()[0] + x.accumulators()[1] for x in (sol, ref)]
    # sums of R (traces: n R) products in FP64 in another order, and of 25 steps: two roundings a term at most
    k = 2 * (len(pairs) + M.n)
    assert np.max(np.abs(tot[0][:k] - tot[1][:k])) <= 2 * (R + 25) * 2.0 ** -53 * np.max(np.abs(tot[1][:k]))
    assert np.max(np.abs(tot[0][k:] - tot[1][k:])) <= 2 * R * M.n * 2.0 ** -53 * np.max(np.abs(tot[1][k:]))
    orc = oracle.OracleRun(M, A, C, h, R, np.concatenate([pairs, fi.diag_pairs(M.n)]), seed=3, burn_in=2,
                           block_len=6).run(25)
    for what, a, b in zip("qps", sol.state(), (orc.q, orc.p, orc.s)):
        if b.size:
            assert np.max(np.abs(a - b)) <= TOL[prec] * np.max(np.abs(b)), what
    both = tot[0][: len(pairs) + M.n], orc.s1 + orc.blk
    assert np.max(np.abs(both[0] - both[1])) <= TOL[prec] * np.max(np.abs(both[1]))


def test_shapes_without_a_kernel_are_refused():
    M = fi.laplacian3d_csr(5, 0.1)
    A, C = random_gle(1, 5)
    sol = fth.Solver(M, A, C, 0.01, replicas=8)
    for shape in ((32, 2, 0), (64, 3, 0), (64, 16, 0), (64, 1, 0)):
        with pytest.raises(fth.FthError) as e:
            fix_shape(sol, *shape)
        assert e.value.status == fth.FTH_EINVAL
    with pytest.raises(fth.FthError) as e:
        fix_shape(fth.Solver(fi.dense_ggt(40, 1), A, C, 0.01, replicas=4), 64, 2, 0)
    assert e.value.status == fth.FTH_EUNSUPPORTED
