"""Measured cases of the f-thermostat library on one GPU.

A case is one solve as a user's program drives it between two looks at its
result: `run(steps)` on a context that is already set up, then `read()`.  The
steps of a pass are one check interval (200 steps is the serving layer's own
default), so a pass holds the step kernels, the schedule around them and the
readout.  One case is the serving layer: a handful of mixed requests from
submission to their results.

Estimates of the FP32 solves are kept in FP32, the precision of the state that
they are formed from; FP64 solves keep FP64.

`exact` integrates the same trajectory in 64 bits with torch: Philox4x32-10
noise, Box-Muller, the half kicks around the exact Ornstein-Uhlenbeck step, the
drift and the block averages, written from the library's header.
"""
import math

import numpy as np
import torch

import fth_inputs as fi
from paper_1402_2095_amd import fth

PRECISION = {"fp64": fth.FTH_FP64, "fp32": fth.FTH_FP32, "bf16x3": fth.FTH_FP32_BF16X3}


# ------------------------------------------------------------------ the cases
def listed():
    """Each case with what it stands for in use."""
    return [
        # the small validation system (single trajectory, white noise, FP64, all of row 0): the
        # smallest call there is, launches and latency count
        _solve("small-64-fp64", "haar", 64, 1, "white", "fp64", 200, pairs=63),
        # a small dense system with a few replicas in FP32: still one workgroup, more work per step
        _solve("small-100-r16", "haar", 100, 16, "invsqrt_ns4", "fp32", 200, pairs=128),
        # a dense request of middling size at the serving layer's replica count, an odd size
        _solve("dense-2100-r64", "dense", 2100, 64, "invsqrt_ns4", "bf16x3", 200, pairs=256),
        # the large dense system of the benchmark
        _solve("dense-16384-r128", "dense", 16384, 128, "invsqrt_ns4", "bf16x3", 100, pairs=1024),
        # a dense system followed with a single trajectory, as the paper runs its examples
        _solve("dense-6001-r1", "dense", 6001, 1, "invsqrt_ns4", "fp32", 200, pairs=1024),
        # the plain FP64 form of a dense system
        _solve("dense-4000-r32-fp64", "dense", 4000, 32, "invsqrt_ns4", "fp64", 100, pairs=1024),
        # the 3-D Laplacian of the benchmark: few replicas, the state fits the cache
        _solve("laplacian-64-r8", "laplacian", 64, 8, "invsqrt_ns4", "fp32", 200, pairs=1024),
        # the banded system of the benchmark: the largest sparse solve
        _solve("banded-1e6-r32", "banded", 1000000, 32, "fermi_b20_ns4", "fp32", 200, pairs=1024),
        # the same kind of system in plain FP64, an odd size
        _solve("banded-250007-r32-fp64", "banded", 250007, 32, "fermi_b20_ns4", "fp64", 100, pairs=1024),
        # occupation of a gapped lattice: momentum-form estimates with six extra momenta
        _solve("insulator-48-r32-pp", "insulator", 48, 32, "fermi_gap_p_ns6", "fp32", 200, pairs=1024, momentum=True),
        # log det of the paper's M1 lattice: 81 entries a row, eight extra momenta, traces
        _solve("m1-24-r32-traces", "m1", 24, 32, "ln_p_ns8", "fp32", 200, pairs=1024, momentum=True, traces=True),
        # mixed requests through the serving layer, from submission to result
        {"name": "serving-mix", "kind": "serving", "requests": 6, "n_sparse": 40000, "n_dense": 900, "steps": 400},
    ]


def draw(rng):
    """One more solve (or mix of requests) of the same ranges."""
    def log_between(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    family = rng.choice(["small", "dense", "dense", "single", "dense64", "laplacian", "banded", "banded64",
                         "insulator", "m1", "serving"])
    pairs = rng.choice([1, 100, 256, 1024])
    if family == "small":
        n, r = rng.choice([(rng.randint(20, 120), 1), (rng.randint(20, 100), 4), (rng.randint(20, 100), 16)])
        return _solve(None, "haar", n, r, rng.choice(["white", "invsqrt_ns4"]), rng.choice(["fp32", "fp64"]),
                      rng.choice([100, 200, 400]), pairs=rng.choice([1, 40, 128]))
    if family == "dense":
        return _solve(None, "dense", log_between(520, 9000), rng.choice([16, 32, 64, 128]), "invsqrt_ns4", "bf16x3", 100,
                      pairs=pairs)
    if family == "single":
        return _solve(None, "dense", log_between(4200, 9000), rng.choice([1, 2, 4, 8]), "invsqrt_ns4",
                      rng.choice(["fp32", "fp32", "fp64"]), 100, pairs=pairs)
    if family == "dense64":
        return _solve(None, "dense", log_between(520, 5000), rng.choice([16, 32, 64]), "invsqrt_ns4", "fp64", 100,
                      pairs=pairs)
    if family == "laplacian":
        return _solve(None, "laplacian", rng.randint(20, 80), rng.choice([4, 8, 16]), "invsqrt_ns4",
                      rng.choice(["fp32", "fp32", "fp64"]), rng.choice([100, 200]), pairs=pairs)
    if family == "banded":
        return _solve(None, "banded", log_between(30000, 900000), rng.choice([8, 16, 32]),
                      rng.choice(["fermi_b20_ns4", "invsqrt_ns4"]), "fp32", rng.choice([100, 200]), pairs=pairs,
                      momentum=rng.random() < 0.3)
    if family == "banded64":
        return _solve(None, "banded", log_between(30000, 250000), rng.choice([8, 16, 32]), "fermi_b20_ns4", "fp64", 100,
                      pairs=pairs)
    if family == "insulator":
        return _solve(None, "insulator", 2 * rng.randint(10, 26), rng.choice([8, 16, 32]),
                      rng.choice(["fermi_gap_p_ns4", "fermi_gap_p_ns6"]), "fp32", rng.choice([100, 200]), pairs=pairs,
                      momentum=True)
    if family == "m1":
        return _solve(None, "m1", rng.randint(10, 26), rng.choice([8, 16, 32]), rng.choice(["ln_p_ns8", "ln_p_ns10"]),
                      "fp32", 100, pairs=pairs, momentum=True, traces=rng.random() < 0.5)
    return {"kind": "serving", "requests": rng.randint(2, 6), "n_sparse": log_between(10000, 40000),
            "n_dense": rng.randint(512, 1000), "steps": 400}


def _solve(name, matrix, n, replicas, gle, precision, steps, pairs, momentum=False, traces=False):
    case = {"kind": "solve", "matrix": matrix, "n": n, "replicas": replicas, "gle": gle, "precision": precision,
            "steps": steps, "pairs": pairs, "momentum": bool(momentum), "traces": bool(traces)}
    return case if name is None else {"name": name, **case}


# ------------------------------------------------------------------ inputs
def _banded(n, seed):
    """fth_inputs.banded_spd_csr's kind of matrix (offsets -3..3, 7 entries a row), laid out directly as CSR."""
    rng = np.random.default_rng(seed)
    offd = [rng.uniform(-1.0, 0.0, size=n).astype(np.float32) for _ in range(3)]  # offd[k-1][i]: (i, i + k)
    slots = np.zeros((n, 7), dtype=np.float32)
    have = np.zeros((n, 7), dtype=bool)
    for k in (1, 2, 3):
        slots[: n - k, 3 + k] = offd[k - 1][: n - k]
        slots[k:, 3 - k] = offd[k - 1][: n - k]
        have[: n - k, 3 + k] = True
        have[k:, 3 - k] = True
    radius = np.abs(slots).sum(axis=1, dtype=np.float64)
    slots[:, 3] = radius + rng.uniform(0.05, 1.0, size=n)
    have[:, 3] = True
    col = np.arange(n, dtype=np.int32)[:, None] + np.arange(-3, 4, dtype=np.int32)[None, :]
    row_ptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(have.sum(axis=1), out=row_ptr[1:])
    return fi.CSR(n, row_ptr, col[have], slots[have]), float(np.max(slots[:, 3] + radius))


def _dense(n, seed, dtype):
    """G G^T / n + 0.1 I, drawn and multiplied on the GPU; its spectrum ends near 4.1."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(n, n, generator=g, device="cuda", dtype=torch.float32).double()
    m = x @ x.T
    m = (m + m.T) / (2.0 * n)
    m.diagonal().add_(0.1)
    return m.to(dtype).cpu().numpy(), 4.4


def _problem(matrix, n, replicas, gle, precision, steps, pairs, seed, momentum=False, traces=False):
    """Everything that defines one solve, as plain values and arrays."""
    fp64 = precision == "fp64"
    if matrix == "haar":
        M, lam = fi.haar_spd(n, seed + 1, 0.1, 12.1)
        lam_max = float(lam.max())
        M = M if fp64 else M.astype(np.float32)
    elif matrix == "dense":
        M, lam_max = _dense(n, seed + 1, torch.float32)
    elif matrix == "laplacian":
        M, lam_max = fi.laplacian3d_csr(n, 0.1), fi.laplacian3d_lambda_max(n, 0.1)
    elif matrix == "banded":
        M, lam_max = _banded(n, seed + 1)
    elif matrix == "insulator":
        M, lam_max = fi.insulator3d_csr(n), 12.1
    elif matrix == "m1":
        M = fi.m1_lattice_csr(n, seed + 1, dtype=np.float32)
        lam_max = fi.gershgorin_max(M)
    else:
        raise ValueError(matrix)
    g = fi.white_noise_gle() if gle == "white" else fi.load_gle(gle)
    rows = M.shape[0] if isinstance(M, np.ndarray) else M.n
    return {"M": M, "rows": rows, "A_p": g.A_p, "C_p": g.C_p, "h": fi.dt_rule(lam_max),
            "pairs": fi.random_pairs(rows, pairs, seed + 2), "replicas": replicas, "precision": precision,
            "seed": 77 + seed, "stream_id": 0, "burn_in": 0, "block_len": 50, "steps": steps, "diag": True,
            "momentum": momentum, "traces": traces, "scale_r": 1.0, "scale_m": 0.0, "invsqrt": False}


def _solve_problem(case, seed):
    return _problem(case["matrix"], case["n"], case["replicas"], case["gle"], case["precision"], case["steps"],
                    case["pairs"], seed, case["momentum"], case["traces"])


def _requests(case, seed):
    """The mixed requests of one serving pass: sparse and dense, x^-1/2 and Fermi targets, each with the
    spectral map that puts its spectrum into the thermostat's window."""
    rng = np.random.default_rng(seed)
    out = []
    for k in range(case["requests"]):
        kind = ("laplacian", "banded", "dense")[k % 3]
        if kind == "laplacian":
            n = max(3, int(round((case["n_sparse"] * rng.uniform(0.5, 1.0)) ** (1 / 3))))
        else:
            n = int(case["n_dense" if kind == "dense" else "n_sparse"] * rng.uniform(0.5, 1.0))
        gle = ("invsqrt_ns4", "fermi_b20_ns4")[(k // 3) % 2]
        p = _problem(kind, n, 64 if kind == "dense" else 32, gle, "bf16x3" if kind == "dense" else "fp32",
                     case["steps"], 1, seed + 1000 * (k + 1))
        lam_hi = (0.1 / p["h"]) ** 2
        w_lo, w_hi = fi.load_gle(gle).meta["window_lambda"]
        if gle == "invsqrt_ns4":
            p.update(scale_r=w_hi / lam_hi, invsqrt=True)
        else:
            r, m = fth.fth_spectral_map(0.05, lam_hi, w_lo, w_hi)
            p.update(scale_r=r, scale_m=m)
        d = rng.choice(p["rows"], size=128, replace=False)
        a = rng.integers(0, 128, size=128)
        b = (a + 1 + rng.integers(0, 127, size=128)) % 128
        p.update(pairs=np.concatenate([np.stack([d, d], 1), np.stack([d[a], d[b]], 1)]).astype(np.int32), diag=False,
                 h=fi.dt_rule(w_hi), stream_id=k + 1, burn_in=100, block_len=100)
        out.append(p)
    return out


# ------------------------------------------------------------------ a pass
def prepare(case, seed):
    if case["kind"] == "serving":
        reqs = [dict(M=p["M"], A_p=p["A_p"], C_p=p["C_p"], dt=p["h"], pairs=p["pairs"], replicas=p["replicas"],
                     precision=PRECISION[p["precision"]], seed=p["seed"], stream_id=p["stream_id"],
                     burn_in=p["burn_in"], block_len=p["block_len"], target=1e-2, max_steps=p["steps"],
                     scale_r=p["scale_r"], scale_m=p["scale_m"],
                     unscale_target=fth.FTH_TARGET_INVSQRT if p["invsqrt"] else -1) for p in _requests(case, seed)]
        return {"case": case, "server": fth.Server(), "requests": reqs}
    p = _solve_problem(case, seed)
    sol = fth.Solver(p["M"], p["A_p"], p["C_p"], p["h"], pairs=p["pairs"], replicas=p["replicas"],
                     precision=PRECISION[p["precision"]], seed=p["seed"], burn_in=p["burn_in"],
                     block_len=p["block_len"], acc_diag=p["diag"], tune=True, acc_pp=p["momentum"],
                     acc_trace=p["traces"])
    sol.run(0)  # fixes the launch shape
    return {"case": case, "solver": sol}


def run(state):
    case = state["case"]
    if case["kind"] == "serving":
        srv = state["server"]
        ids = [srv.submit(**r) for r in state["requests"]]
        live = list(ids)
        while live:
            srv.tick()
            live = [i for i in live if srv.poll(i)["state"] < fth.FTH_REQ_DONE]
        return [_parts(*(x.astype(np.float32) for x in srv.result(i))) for i in ids]
    sol = state["solver"]
    est, se, _ = sol.run(case["steps"]).read()
    if case["precision"] != "fp64":
        est, se = est.astype(np.float32), se.astype(np.float32)
    return _parts(est, se, case)


def _parts(est, se, case=None):
    """The estimates by kind: position form, momentum form, traces."""
    out = {"qq": est, "qq_se": se}
    if case is None or not (case["momentum"] or case["traces"]):
        return out
    ntr = (3 if case["momentum"] else 2) if case["traces"] else 0
    each = (len(est) - ntr) // (2 if case["momentum"] else 1)
    out = {"qq": est[:each], "qq_se": se[:each]}
    if case["momentum"]:
        out.update(pp=est[each: 2 * each], pp_se=se[each: 2 * each])
    if ntr:
        out.update(traces=est[-ntr:], traces_se=se[-ntr:])
    return out


# ------------------------------------------------------------------ figures
CHIP_BYTES = 256 << 20  # the last-level cache: a matrix beyond it comes from memory in every step


def _sizes(case):
    n = case["n"]
    rows = n ** 3 if case["matrix"] in ("laplacian", "insulator", "m1") else n
    nnz = {"haar": rows * rows, "dense": rows * rows, "m1": 81 * rows}.get(case["matrix"], 7 * rows)
    ns = 0 if case["gle"] == "white" else fi.load_gle(case["gle"]).ns
    return rows, nnz, ns


def work(case):
    """Matrix, state and accumulators in and out once per pass (a dense matrix larger than the last-level cache
    once per step); the products, the thermostat's FMAs, ten operations a normal and the sampled squares of every
    step."""
    if case["kind"] == "serving":
        total = {"bytes": 0.0, "flops": 0.0}
        for k in range(case["requests"]):
            kind = ("laplacian", "banded", "dense")[k % 3]
            n = 0.75 * case["n_dense" if kind == "dense" else "n_sparse"]
            w = work(_solve(None, "dense" if kind == "dense" else "banded", n, 64 if kind == "dense" else 32,
                            "invsqrt_ns4", "fp32", case["steps"], 256))
            total = {x: total[x] + w[x] for x in total}
        return total
    rows, nnz, ns = _sizes(case)
    real = 8.0 if case["precision"] == "fp64" else 4.0
    dense = case["matrix"] in ("haar", "dense")
    matrix = nnz * real if dense else nnz * (real + 4.0) + 4.0 * rows
    times = case["steps"] if dense and matrix > CHIP_BYTES else 1
    kinds = 2.0 if case["momentum"] else 1.0
    state = 2.0 * rows * case["replicas"] * (ns + 2) * real
    acc = kinds * (rows + case["pairs"]) * (2 * 24.0 + 16.0)
    d = ns + 1
    per_dof = 2.0 * (d * d + d * (d + 1) / 2) + 10.0 * d + 6.0 + 2.0 * kinds
    return {"bytes": float(times * matrix + state + acc),
            "flops": float(case["steps"]) * case["replicas"] * (2.0 * nnz + rows * per_dof)}


# ------------------------------------------------------------------ 64 bits
def exact(case, seed):
    if case["kind"] == "serving":
        return [_parts(*_integrate(p)) for p in _requests(case, seed)]
    return _parts(*_integrate(_solve_problem(case, seed)), case)


def _philox(c0, c1, c2, c3, key):
    """Philox4x32-10 on int64 tensors that hold 32-bit words (products wrap, the masks keep the words)."""
    low = 0xFFFFFFFF
    k0, k1 = key & low, (key >> 32) & low
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c2 = ((b >> 32) & low) ^ c1 ^ k0, ((a >> 32) & low) ^ c3 ^ k1
        c1, c3 = b & low, a & low
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return c0, c1, c2, c3


def _normals(p, n, comps, dev):
    """xi[component, row, replica] of step n."""
    groups = (p["replicas"] + 3) // 4
    i = torch.arange(p["rows"], device=dev, dtype=torch.int64).view(1, -1, 1)
    r = torch.arange(groups, device=dev, dtype=torch.int64).view(1, 1, -1)
    j = torch.arange(comps, device=dev, dtype=torch.int64).view(-1, 1, 1)
    shape = (comps, p["rows"], groups)
    words = _philox(i.expand(shape), torch.tensor(n, device=dev), ((j << 16) | r).expand(shape),
                    torch.tensor(p["stream_id"], device=dev), p["seed"])
    u = [(2.0 * (w >> 9).double() + 1.0) * 2.0 ** -24 for w in words]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        radius = torch.sqrt(-2.0 * torch.log(a))
        z += [radius * torch.cos(2.0 * math.pi * b), radius * torch.sin(2.0 * math.pi * b)]
    return torch.stack(z, dim=-1).reshape(comps, p["rows"], 4 * groups)[:, :, : p["replicas"]].contiguous()


def _force_of(p, dev):
    """A function that gives M' q for M' = r M + m I in 64 bits."""
    M, r, m = p["M"], p["scale_r"], p["scale_m"]
    if isinstance(M, np.ndarray):
        D = torch.from_numpy(M).to(dev).double() * r
        D.diagonal().add_(m)
        return lambda q: D @ q
    counts = np.diff(M.row_ptr)
    width = int(counts.max())
    at = np.arange(len(M.col)) - np.repeat(M.row_ptr[:-1], counts)
    rows = np.repeat(np.arange(M.n), counts)
    col = np.zeros((width, M.n), dtype=np.int64)
    val = np.zeros((width, M.n))
    col[at, rows] = M.col
    val[at, rows] = M.val.astype(np.float64) * r + np.where(M.col == rows, m, 0.0)
    col, val = torch.from_numpy(col).to(dev), torch.from_numpy(val).to(dev).unsqueeze(-1)

    def force(q):
        out = val[0] * q[col[0]]
        for u in range(1, width):
            out.addcmul_(val[u], q[col[u]])
        return out

    return force


def _integrate(p):
    """Estimates and standard errors of one solve from its start, all in 64 bits."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    rows, R, h = p["rows"], p["replicas"], p["h"]
    comps = p["A_p"].shape[0]
    A, C = torch.from_numpy(np.array(p["A_p"])).double(), torch.from_numpy(np.array(p["C_p"])).double()
    T = torch.linalg.matrix_exp(-A * h)
    S = torch.linalg.cholesky(C - T @ C @ T.T).tolist()
    T = T.tolist()
    mul = _force_of(p, dev)
    q = torch.zeros(rows, R, device=dev, dtype=torch.float64)
    x = torch.zeros(comps, rows, R, device=dev, dtype=torch.float64)
    pairs = torch.from_numpy(p["pairs"].astype(np.int64)).to(dev)

    def sample(v):
        some = (v[pairs[:, 0]] * v[pairs[:, 1]]).sum(1)
        return torch.cat([some, (v * v).sum(1)]) if p["diag"] else some

    block = s1 = s2 = 0.0
    done = 0
    for n in range(p["steps"]):
        mq = mul(q)
        if n >= p["burn_in"]:
            parts = [sample(q)] + ([sample(x[0])] if p["momentum"] else [])
            if p["traces"]:
                parts.append(torch.stack([(q * q).sum(), (q * mq).sum()] +
                                         ([(x[0] * x[0]).sum()] if p["momentum"] else [])))
            block = block + torch.cat(parts)
            done += 1
            if done % p["block_len"] == 0:
                s1, s2, block = s1 + block, s2 + block * block, torch.zeros_like(block)
        xi = _normals(p, n, comps, dev)
        x[0] -= 0.5 * h * mq
        y = torch.empty_like(x)
        for r in range(comps):
            y[r] = T[r][0] * x[0]
            for c in range(1, comps):
                y[r].add_(x[c], alpha=T[r][c])
            for c in range(r + 1):
                y[r].add_(xi[c], alpha=S[r][c])
        y[0] -= 0.5 * h * mq
        x = y
        q = q + h * x[0]
    blocks = done // p["block_len"]
    est = (s1 + block) / (R * done)
    scale = 1.0 / (R * p["block_len"])
    var = (s2 * scale * scale - (s1 * scale) ** 2 / blocks) / (blocks - 1)
    se = torch.sqrt(var.clamp_min(0.0) / blocks)
    if p["invsqrt"]:
        est, se = est * math.sqrt(p["scale_r"]), se * math.sqrt(p["scale_r"])
    return est.cpu().numpy(), se.cpu().numpy()
