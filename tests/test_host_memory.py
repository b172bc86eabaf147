"""Host memory that runs out inside an init call comes back as PDBO_ENOMEM; no
exception leaves the C entry points."""
import os
import subprocess
import sys

import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROG = r"""
import ctypes, resource, sys
import numpy as np
from paper_2509_21064_amd import _abi
lib = _abi.load()
par = _abi.pdbo_params(B=4, eval_every=1, alpha=0.01, beta=0.01, y0=1.0, delta=0.01, scale=1.0, g_degree=1)
ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
ctx = ctypes.c_void_p()
if sys.argv[1] == "maxsat":
    m, n, k = 4000000, 5000, 5
    lits = (np.arange(m * k, dtype=np.int32).reshape(m, k) % n) + 1
    prob = _abi.pdbo_maxsat(n=n, m=m, k=k, lits=ptr(lits))
    init = lib.maxsat_gda_init
else:
    n, d = 4000, 1000
    rp = np.arange(n + 1, dtype=np.int32) * d
    col = np.tile(np.arange(d, dtype=np.int32), n)
    val = np.ones(n * d, np.int32)
    prob = _abi.pdbo_qubo(n=n, format=1, row_ptr=ptr(rp), col_idx=ptr(col), q=ptr(val), nnz=n * d)
    init = lib.qubo_gda_init
used = int(next(l for l in open("/proc/self/status") if l.startswith("VmSize")).split()[1]) << 10
resource.setrlimit(resource.RLIMIT_AS, (used + (32 << 20), resource.RLIM_INFINITY))
status = init(ctypes.byref(prob), ctypes.byref(par), None, ctypes.byref(ctx))
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
print("status", status, bool(ctx))
"""


@pytest.mark.parametrize("kind", ["maxsat", "csr"])
def test_host_allocation_failure_is_a_status(kind):
    """Before any device call (runs without a GPU)."""
    r = subprocess.run([sys.executable, "-c", PROG, kind], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    assert r.stdout.split()[-3:] == ["status", "2", "False"], r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["dense", "csr", "csr_many", "rows", "split", "maxsat", "kcut"])
def test_host_allocation_failure_frees_the_device(kind, monkeypatch):
    import torch
    from gpu_util import require_gpu, say
    P = require_gpu()
    if kind == "dense":
        q = W.random_dense_qubo(300, -50, 50, W.rng_for(3, 46, 0, 300))
        mk = lambda: P.qubo_gda_init(q, W.gda_params("qubo", B=16, T=1, scale=50.0), None)
    elif kind == "maxsat":
        f = W.random_maxsat(300, 1200, 3, 1, 10, W.rng_for(5, 46, 0))
        mk = lambda: P.maxsat_gda_init(f, W.gda_params("maxsat", B=16, T=1, scale=5.5), None)
    elif kind == "kcut":
        g = W.kcut_graph(400, 1200, 3, rep=1)
        mk = lambda: P.kcut_gda_init(g, dict(B=8, T=1, alpha=0.01, beta=0.01, y0=0.5, delta=2.0 ** -7, scale=1.0,
                                             g="quad", seed=3), None)
    else:
        q = W.maxcut_c2(0, n=400, M=1200)
        if kind == "split":
            monkeypatch.setenv("PDBO_CSR_SPLIT", "1")
        p = W.gda_params("maxcut", B=130 if kind == "csr_many" else 8, T=1, tile=0 if kind.startswith("csr") else 2)
        mk = lambda: P.qubo_gda_init(q, p, None)
    mk().destroy()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    failures = 0
    monkeypatch.setenv("PDBO_FAIL_ALLOC_HOST", "1")
    for k in (1, 2, 3, 5, 8, 13, 21):
        say(f"[host memory] {kind} at allocation {k}")
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", str(k))
        try:
            mk().destroy()
        except P.PdboError as e:
            assert e.status == 2, e
            failures += 1
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", "0")
        assert torch.cuda.mem_get_info()[0] >= free0 - (2 << 20), k
    assert failures >= 4
    mk().destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["csr", "csr_many", "split", "kcut"])
@pytest.mark.parametrize("host", [False, True])
def test_no_room_for_the_layout(kind, host, monkeypatch):
    """The layouts of csr_resident, csr_split and kcut_resident are optional: an
    allocation of theirs that fails, on the device or the host, leaves the context
    on the kernels it would otherwise run on, with the same run."""
    import numpy as np
    from gpu_util import require_gpu, say
    P = require_gpu()
    if kind == "kcut":
        g = W.kcut_graph(400, 1200, 3, rep=1)
        mk = lambda: P.kcut_gda_init(g, dict(B=8, T=1, alpha=0.01, beta=0.01, y0=0.5, delta=2.0 ** -7, scale=1.0,
                                             g="quad", seed=3), None)
    else:
        if kind == "split":
            monkeypatch.setenv("PDBO_CSR_SPLIT", "1")
        q = W.maxcut_c2(0, n=400, M=1200)
        p = W.gda_params("maxcut", B=130 if kind == "csr_many" else 8, T=1, tile=2 if kind == "split" else 0, seed=5)
        mk = lambda: P.qubo_gda_init(q, p, None)
    # allocations of the layout, and what the context runs on with and without it
    parts, names = {"csr": (5, ("csr_resident_seq", "csr_rows")), "csr_many": (3, ("csr_resident", "csr_packed_dbuf_t32")),
                    "split": (3, ("csr_split", "csr_rows")), "kcut": (8, ("", ""))}[kind]

    def run():
        ctx = mk()
        name = ctx.tile_name
        ctx.step(30)
        r = ctx.result()
        out = [*ctx.get_state()[:2], ctx.objectives(), r["best_obj"], r["best_x"]]
        ctx.destroy()
        return name, out

    name, ref = run()
    assert name == names[0]
    if host:
        monkeypatch.setenv("PDBO_FAIL_ALLOC_HOST", "1")
    refused, fell_back = [], 0
    for k in range(1, 40):
        say(f"[no room] {kind} allocation {k} host={host}")
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", str(k))
        try:
            name, got = run()
            fell_back += name == names[1]
            for a, b in zip(got, ref):
                assert np.array_equal(a, b)
        except P.PdboError as e:
            assert e.status == 2
            refused.append(k)
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", "0")
    assert max(refused) - len(refused) == parts
    assert kind == "kcut" or fell_back == parts
