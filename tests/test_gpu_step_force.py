"""The force inside a dense step, not the one of fth_force (which some contexts
form with another kernel): one step from a state whose kicks outweigh the noise
shows it in the momenta.  From p = s = 0 and q given, the step is
p' = T_00 k + (S xi)_0 + k with the half kick k = -h/2 M q, s'_c = T_c0 k + (S xi)_c."""
import numpy as np
import pytest

import fth_inputs as fi
import oracle
from paper_1402_2095_amd import fth

pytestmark = pytest.mark.gpu

SPLIT, F32, F64 = fth.FTH_FP32_BF16X3, fth.FTH_FP32, fth.FTH_FP64


@pytest.mark.parametrize("n, R, prec, name", [
    (257, 16, SPLIT, "dense_rows_bf16x3_kernel<NS=4,CT=1>"),
    (513, 64, SPLIT, "dense_rows_bf16x3_kernel<NS=4,CT=1>"),
    (520, 128, SPLIT, "dense_rows_bf16x3_kernel<NS=4,CT=2>"),
    (1571, 128, SPLIT, "dense_rows_bf16x3_kernel<NS=4,CT=4>"),
    (2111, 16, SPLIT, "dense_rows_bf16x3_kernel<NS=4,CT=1>"),
    (2310, 64, SPLIT, "gemm_bf16x3_kernel"),
    (271, 16, F64, "dense_rows_f64_kernel<NS=4,CT=1>"),
    (560, 128, F64, "dense_rows_f64_kernel<NS=4,CT=2>"),
    (1260, 64, F64, "gemm_f64_kernel"),    # K slices of 16 and 15 k-steps
    (1280, 64, F64, "gemm_f64_kernel"),    # all of 16
    (2559, 32, F64, "gemm_f64_kernel"),    # all of 20, the last k-step not full
    (4099, 1, F32, "dense_gemv_kernel"),
    (515, 8, F64, "dense_gemv_kernel"),
    (100, 16, F32, "small_dense_kernel_quad"),
    (127, 4, F64, "small_dense_kernel_quad"),
    (250, 4, F64, "small_dense_kernel<"),
])
def test_force_of_a_step(n, R, prec, name):
    M = fi.dense_ggt(n, 3 + n)
    M64 = M.astype(np.float64)
    h = fi.dt_rule(fi.power_lambda_max(M64))
    g = fi.load_gle("invsqrt_ns4")
    sol = fth.Solver(M, g.A_p, g.C_p, h, replicas=R, precision=prec, seed=3, stream_id=2)
    assert sol.kernel_name.startswith(name), sol.kernel_name
    q = (1e5 * np.random.default_rng(n).normal(size=(n, R))).astype(np.float32).astype(np.float64)
    sol.set_state(q=q, p=np.zeros((n, R)), s=np.zeros((sol.ns, n, R)))
    sol.run(1)
    _, p, s = sol.state()

    T, S = fth.fth_propagator(g.A_p, g.C_p, h)
    d = sol.ns + 1
    i, r = np.meshgrid(np.arange(n), np.arange(R), indexing="ij")
    xi = np.stack([oracle.normals(3, 2, i.ravel(), r.ravel(), 0, c).reshape(n, R) for c in range(d)])
    kick = -0.5 * h * (M64 @ q)
    z = np.einsum("cd,dir->cir", S, xi) + T[:, 0][:, None, None] * kick
    z[0] += kick
    # The force's own bound (fth_force's against an FP64 product) and eight roundings of the update; the momenta
    # hold up to twice the half kick.
    tol = {SPLIT: 3e-5, F32: 3e-5, F64: 1e-13}[prec] + 8 * 2.0 ** (-53 if prec == F64 else -24)
    scale = np.max(np.abs(kick))
    assert scale > 200 * np.max(np.abs(xi))
    for what, a, b in (("p", p, z[0]), ("s", s, z[1:])):
        assert np.max(np.abs(a - b)) <= 2 * tol * scale, (what, np.max(np.abs(a - b)) / scale)
