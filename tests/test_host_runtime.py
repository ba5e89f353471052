"""The library's host code against a HIP runtime without a device
(host_runtime.cpp, CPU): the order of its work on streams, its memory and its
failure paths.  Each case runs in a child process that loads the stand-in
runtime before the library; kernels are recorded, not run, so no result of a
solve is looked at here."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

VERSIONS = """
hip_4.2 { global: hip*; __hip*; stub_*; };
hip_4.3 { global: hipGraphDestroy; hipGraphExecDestroy; hipGraphInstantiate; hipGraphLaunch;
                  hipStreamBeginCapture; hipStreamEndCapture; } hip_4.2;
"""

PRELUDE = """
import ctypes, os
stub = ctypes.CDLL(os.environ["FTH_TEST_RUNTIME"], mode=ctypes.RTLD_GLOBAL)
for name, res, args in (("stub_live", ctypes.c_size_t, []), ("stub_peak", ctypes.c_size_t, []),
                        ("stub_live_on", ctypes.c_size_t, [ctypes.c_int]),
                        ("stub_host_live", ctypes.c_size_t, []), ("stub_limit", None, [ctypes.c_size_t]),
                        ("stub_devices", None, [ctypes.c_int]),
                        ("stub_fail_in", None, [ctypes.c_long]), ("stub_mallocs", ctypes.c_long, []),
                        ("stub_frees", ctypes.c_long, []), ("stub_launches", ctypes.c_long, []),
                        ("stub_violations", ctypes.c_long, []), ("stub_violation", ctypes.c_char_p, [ctypes.c_long]),
                        ("stub_logged", ctypes.c_long, []), ("stub_kernel", ctypes.c_char_p, [ctypes.c_long]),
                        ("stub_reset", None, [])):
    f = getattr(stub, name)
    f.restype, f.argtypes = res, args
import numpy as np
import fth_inputs as fi
from paper_1402_2095_amd import fth
g = fi.load_gle("invsqrt_ns4")
def no_violations():
    v = [stub.stub_violation(k).decode() for k in range(stub.stub_violations())]
    assert not v, (len(v), sorted(set(v))[:6])
def kernels():
    return [stub.stub_kernel(k).decode() for k in range(stub.stub_logged())]
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_runtime")
    script, out = d / "versions", d / "libamdhip64.so.7"
    script.write_text(VERSIONS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                    f"-Wl,--version-script={script}", os.path.join(ROOT, "tests", "host_runtime.cpp"), "-o", str(out)],
                   check=True)
    return str(out)


def run_child(runtime, code):
    env = dict(os.environ, FTH_TEST_RUNTIME=runtime, PYTHONPATH=ROOT)
    res = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(code) + "\nprint('child ok')"], env=env,
                         capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert res.returncode == 0 and "child ok" in res.stdout, (res.stdout + res.stderr)[-4000:]


SYSTEMS = """
def systems():
    M = fi.banded_spd_csr(700, 3)
    D = fi.dense_ggt(700, 3)
    S = fi.dense_ggt(60, 3)
    for late in (False, True):   # the replica count given at create, or at the first run
        yield M, 32, fth.FTH_FP32, late
        yield M, 8, fth.FTH_FP64, late
        yield S, 4, fth.FTH_FP64, late
        yield D, 8, fth.FTH_FP32, late
        yield D, 64, fth.FTH_FP32_BF16X3, late
        yield fi.dense_ggt(2300, 3), 64, fth.FTH_FP32_BF16X3, late
        yield D, 16, fth.FTH_FP64, late
"""


@pytest.mark.parametrize("trace", [0, 1])
@pytest.mark.parametrize("tune", [0, 1])
def test_work_waits_for_the_fills_it_needs(runtime, tune, trace):
    """Buffers that start at zero (accumulators, step counter, state, trace
    partials, a force call's scratch) are zero before a kernel runs."""
    run_child(runtime, SYSTEMS + f"""
for M, R, prec, late in systems():
    kw = dict(pairs=fi.random_pairs(60, 20, 1), precision=prec, acc_diag=True, acc_pp=True, acc_trace=bool({trace}),
              tune=bool({tune}))
    sol = fth.Solver(M, g.A_p, g.C_p, 0.01, replicas=0 if late else R, **kw)
    sol.run(70, R)
    sol.read()
    image = sol.save()
    if prec != fth.FTH_FP32 and "quad" not in sol.kernel_name or "gemv" in sol.kernel_name:
        if isinstance(M, np.ndarray):
            sol.force(np.zeros((M.shape[0], R)))
    sol.load(image)
    sol.run(3)
    sol.close()
    no_violations()
assert stub.stub_launches() > 1000
""")


@pytest.mark.parametrize("prec", ["FTH_FP32", "FTH_FP64"])
def test_served_requests_wait_for_their_fills(runtime, prec):
    run_child(runtime, f"""
M = fi.banded_spd_csr(700, 3)
srv = fth.Server(steps_per_tick=20)
ids = [srv.submit(M=M, A_p=g.A_p, C_p=g.C_p, dt=0.01, pairs=fi.random_pairs(700, 20, 1), replicas=32,
                  precision=fth.{prec}, seed=k, target=1e-9, max_steps=60) for k in range(3)]
for _ in range(40):
    srv.tick()
assert all(srv.poll(i)["state"] == fth.FTH_REQ_DONE for i in ids)
srv.close()
no_violations()
""")


@pytest.mark.parametrize("kind", ["create", "run"])
def test_a_failed_allocation_leaves_nothing_behind(runtime, kind):
    """Whichever device allocation of a context fails, the call reports it,
    holds what it held before, and the next call allocates everything: no
    kernel is launched on a buffer that is not there."""
    run_child(runtime, SYSTEMS + f"""
kind = {kind!r}
for M, R, prec, late in systems():
    if late != (kind == "run"):
        continue
    blocked = not isinstance(M, np.ndarray) and prec == fth.FTH_FP32
    kw = dict(pairs=fi.random_pairs(60, 20, 1), precision=prec, acc_diag=True, acc_pp=True, acc_trace=True,
              temporal_steps=3 if blocked else 0)
    sol = fth.Solver(M, g.A_p, g.C_p, 0.01, replicas=0 if late else R, **kw)
    sol.run(10, R)
    want, name = sol.device_bytes, sol.kernel_name
    sol.close()
    k = 0
    while True:
        live = stub.stub_live()
        if kind == "create":
            stub.stub_fail_in(k)
            try:
                sol = fth.Solver(M, g.A_p, g.C_p, 0.01, replicas=R, **kw)
                stub.stub_fail_in(-1)
                break
            except fth.FthError as e:
                assert e.status == fth.FTH_ENOMEM, e
            assert stub.stub_live() == live
        else:
            sol = fth.Solver(M, g.A_p, g.C_p, 0.01, **kw)
            held = sol.device_bytes
            stub.stub_fail_in(k)
            try:
                sol.run(10, R)
                stub.stub_fail_in(-1)
                break
            except fth.FthError as e:
                assert e.status == fth.FTH_ENOMEM, e
            assert sol.device_bytes == held or k >= 4   # or: the state is there, a later buffer is not
            # another replica count is open to a context without a state
            if sol.device_bytes == held and k % 3 == 0 and R != 16 and prec != fth.FTH_FP32:
                sol.run(10, 16)
            else:
                sol.run(10, R)
                assert (sol.device_bytes, sol.kernel_name) == (want, name), (k, sol.device_bytes, want, sol.kernel_name)
            sol.close()
            assert stub.stub_live() == live
        k += 1
    assert k >= 5, k
    sol.close()
    assert stub.stub_live() == live
""")


SERVING = """
def serve(srv, sizes, steps=60, prec=fth.FTH_FP32, R=32, until=fth.FTH_REQ_DONE, A=g.A_p, C=g.C_p):
    ids = [srv.submit(M=fi.banded_spd_csr(n, 3), A_p=A, C_p=C, dt=0.01, pairs=fi.random_pairs(n, 20, 1),
                      replicas=R, precision=prec, seed=n, target=1e-9, max_steps=steps) for n in sizes]
    for _ in range(400):
        srv.tick()
        if all(srv.poll(i)["state"] >= fth.FTH_REQ_DONE for i in ids):
            break
    states = [srv.poll(i)["state"] for i in ids]
    assert states == [until] * len(ids), states
"""


@pytest.mark.parametrize("budget_mb", [44, 64])
def test_server_memory_stays_within_its_budget(runtime, budget_mb):
    """What a server holds for running requests and keeps of finished ones is
    within hbm_budget; without a budget to speak of it keeps at most 1 GiB."""
    run_child(runtime, SERVING + f"""
budget = {budget_mb} << 20
extra = 1 << 20   # the work list of the packed group, rounding of requests
srv = fth.Server(hbm_budget=budget, steps_per_tick=20, max_active=4)
base = stub.stub_live()
rng = np.random.default_rng(1)
for k in range(12):
    sizes = rng.integers(3000, 13000, 5)
    for prec in (fth.FTH_FP32, fth.FTH_FP64):
        serve(srv, sizes, prec=prec)
    assert stub.stub_peak() - base <= budget + extra, (k, stub.stub_peak() - base, budget)
    assert srv.stats()[2] == 0
m = stub.stub_mallocs()
serve(srv, sizes)
serve(srv, sizes)
assert stub.stub_mallocs() - m <= 5 * 16   # what the first of the two took serves the second
srv.close()
assert stub.stub_live() == base and stub.stub_host_live() == 0
no_violations()
""")


def test_server_keeps_a_bounded_amount(runtime):
    run_child(runtime, SERVING + """
srv = fth.Server(steps_per_tick=20, max_active=2)
for n in (130000, 260000, 520000):
    serve(srv, [n], prec=fth.FTH_FP64)
    assert stub.stub_live() <= (1 << 30) + (1 << 20), (n, stub.stub_live())
assert stub.stub_live() > 1 << 28
for n in range(200, 1400):   # many small sizes: the list of known blocks is bounded too
    serve(srv, [n], steps=20, R=4)
srv.close()
assert stub.stub_live() == 0
no_violations()
""")


@pytest.mark.parametrize("first", ["context", "group"])
def test_an_allocation_that_fails_takes_idle_memory_back(runtime, first):
    """Contexts and packed groups alike: a request is not refused for memory
    that the server merely keeps."""
    run_child(runtime, SERVING + f"""
srv = fth.Server(steps_per_tick=20)
if {first!r} == "context":   # idle memory of sizes that do not serve the next request
    serve(srv, [40000], prec=fth.FTH_FP64)
    stub.stub_limit(stub.stub_live() + (1 << 20))
    serve(srv, [50000])
else:   # idle blocks serve the request's context; the work list of its group (one per ns) is not there yet
    serve(srv, [9000, 9000])
    stub.stub_limit(stub.stub_live())
    serve(srv, [9000], A=0.5 * np.eye(4), C=np.eye(4))
assert stub.stub_live() > 0
srv.close()
assert stub.stub_live() == 0
no_violations()
""")


@pytest.mark.parametrize("momentum", [False, True])
def test_a_request_holds_no_more_than_its_footprint(runtime, momentum):
    run_child(runtime, f"""
for M, R, prec in ((fi.banded_spd_csr(3000, 3), 32, fth.FTH_FP32), (fi.banded_spd_csr(3000, 3), 8, fth.FTH_FP64),
                   (fi.dense_ggt(128, 3), 32, fth.FTH_FP64), (fi.dense_ggt(128, 3), 32, fth.FTH_FP32),
                   (fi.dense_ggt(31, 3), 64, fth.FTH_FP32), (fi.dense_ggt(31, 3), 128, fth.FTH_FP64),
                   (fi.dense_ggt(300, 3), 8, fth.FTH_FP64), (fi.dense_ggt(300, 3), 16, fth.FTH_FP32_BF16X3),
                   (fi.dense_ggt(2300, 3), 64, fth.FTH_FP32_BF16X3), (fi.dense_ggt(1100, 3), 4, fth.FTH_FP32)):
    n = M.shape[0] if isinstance(M, np.ndarray) else M.n
    opt = dict(pairs=fi.random_pairs(n, 200, 1), replicas=R, precision=prec)
    sol = fth.Solver(M, g.A_p, g.C_p, 0.01, acc_pp={momentum}, coded_matrix=-1, **opt)
    held = sol.device_bytes
    srv = fth.Server(steps_per_tick=20)
    i = srv.submit(M=M, A_p=g.A_p, C_p=g.C_p, dt=0.01, target=1e-9, max_steps=600, momentum_form={momentum}, **opt)
    # (fills of 256 bytes for arrays without elements are the only rounding)
    assert held <= srv.poll(i)["footprint"] + 1024, (n, R, prec, held, srv.poll(i)["footprint"])
    srv.close()
    sol.close()
""")


def test_the_device_of_a_context_and_of_its_caller(runtime):
    """A context works on the device it was created on, whichever is current
    later, and reading its results leaves the caller's device current."""
    run_child(runtime, SYSTEMS + """
hip = ctypes.CDLL("libamdhip64.so.7")
def current():
    d = ctypes.c_int()
    hip.hipGetDevice(ctypes.byref(d))
    return d.value
for M, R, prec, late in systems():
    assert hip.hipSetDevice(0) == 0
    sol = fth.Solver(M, g.A_p, g.C_p, 0.01, pairs=fi.random_pairs(60, 20, 1), precision=prec, acc_trace=True,
                     replicas=0 if late else R)
    assert hip.hipSetDevice(1) == 0
    sol.run(70, R)          # lays the state out when the replica count comes with the run
    no_violations()
    assert stub.stub_live_on(1) == 0
    hip.hipSetDevice(1)
    sol.read()
    assert current() == 1
    image = sol.save()
    hip.hipSetDevice(0)
    twin = fth.Solver(M, g.A_p, g.C_p, 0.01, pairs=fi.random_pairs(60, 20, 1), precision=prec, acc_trace=True)
    hip.hipSetDevice(1)
    twin.load(image)        # so does loading an image
    assert current() == 1 and stub.stub_live_on(1) == 0
    twin.close()
    sol.close()
    no_violations()
""")


def test_a_request_ends_before_step_2_to_the_32(runtime):
    """Where fth_run refuses to go on: the noise counters would repeat."""
    run_child(runtime, """
M = fi.dense_ggt(129, 3)
srv = fth.Server(steps_per_tick=1 << 30, quantum_ms=-1.0)
i = srv.submit(M=M, A_p=g.A_p, C_p=g.C_p, dt=0.01, pairs=fi.random_pairs(129, 2, 1), replicas=4, precision=fth.FTH_FP64,
               target=1e-30)
for tick in range(4):
    srv.tick()
    if srv.poll(i)["state"] == fth.FTH_REQ_DONE:
        break
assert srv.poll(i)["state"] == fth.FTH_REQ_DONE and srv.poll(i)["steps"] == 3 << 30, srv.poll(i)
""")


def test_validation_needs_no_host_memory_to_speak_of(runtime):
    """A matrix that is there can be checked, also where no further array of
    its rows' size fits the address space: the call goes on to its next step
    (here, to find that there is no device) instead of ending the process."""
    run_child(runtime, """
import resource
n = 10_000_000   # 80 MB of 64-bit cursors: never from the heap's free space
val = np.full(3 * n, -1.0, dtype=np.float32)
M = fi.CSR(n, np.zeros(n + 1, dtype=np.int64), np.zeros(3 * n - 2, dtype=np.int32), val[: 3 * n - 2])
i = np.arange(n, dtype=np.int64)
M.row_ptr[1:] = 3 * (i + 1) - 1
M.row_ptr[n] = 3 * n - 2
M.col[0:2] = (0, 1)
M.col[2:] = (np.repeat(i[1:], 3) + np.tile([-1, 0, 1], n - 1))[: 3 * n - 4]
M.val[0] = 3.0
M.val[3::3] = 3.0
del i
stub.stub_devices(0)
def status(m):
    try:
        fth.fth_create(m, [[1.0]], [[1.0]], 0.05, None, fth.fth_default_options())
    except fth.FthError as e:
        return e.status, str(e)
assert status(M)[0] == fth.FTH_EDEVICE, status(M)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (12 << 20), resource.RLIM_INFINITY))
assert status(M)[0] == fth.FTH_EDEVICE, status(M)
M.val[1] = -1.5
assert status(M)[0] == fth.FTH_EINVAL and "not symmetric at (0, 1)" in status(M)[1], status(M)
M.val[1] = -1.0
M.col[4] = 7
assert status(M)[0] == fth.FTH_EINVAL and "pattern not symmetric at (1, 7)" in status(M)[1], status(M)
""")


def test_torch_memory_is_handed_on_when_its_stream_has_drained(monkeypatch):
    """A block of PyTorch's caching allocator may still be in use by work
    queued on its stream; the library uses it on other streams."""
    import torch
    from paper_1402_2095_amd import fth
    events = []

    class Stream:
        def synchronize(self):
            events.append("drained")

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", lambda n: events.append("taken") or 4096)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream())
    assert fth.torch_allocator().alloc(100, None) == 4096
    assert events == ["taken", "drained"]
