"""The resident kernel over positions against the kernels whose runs it stands
in for: the row-parallel path (few restarts, automatic choice) and the CSR-order
resident kernel (PDBO_CSR_SLICED=0).  The sums are the same in the same order
and the objectives are integers, so everything is compared bit for bit."""
import numpy as np
import pytest

import workloads as W
from gpu_util import require_gpu, say
from oracle import qubo as oq

pytestmark = pytest.mark.gpu


def _graph(n, deg, seed, wmax=1, hub=0, even=False):
    """Random symmetric-in-effect QUBO: about n deg / 2 entries stored once or
    twice, a diagonal, c, rows without entries and (hub) one long row."""
    g = np.random.default_rng([n, deg, seed])
    m = max(0, n * deg // 2)
    i, j = g.integers(0, n, m), g.integers(0, n, m)
    if hub:
        k = min(hub, n - 1)
        i, j = np.concatenate([i, np.zeros(k, np.int64)]), np.concatenate([j, g.permutation(n - 1)[:k] + 1])
    keys, first = np.unique(i * n + j, return_index=True)
    i, j = i[first], j[first]
    keep = (i % 7 != 3) & (j % 7 != 3)  # rows without entries
    i, j = i[keep], j[keep]
    v = g.integers(1, wmax + 1, len(i)) * g.choice([-1, 1], len(i))
    if even:  # both triangles: kappa = 2
        up = i < j
        i, j, v = np.concatenate([i[up], j[up]]), np.concatenate([j[up], i[up]]), np.concatenate([v[up], v[up]])
    order = np.lexsort((j, i))
    rp = np.zeros(n + 1, np.int64)
    np.add.at(rp, i + 1, 1)
    return W.Qubo(n=n, row_ptr=np.cumsum(rp).astype(np.int32), col_idx=j[order].astype(np.int32),
                  vals=v[order].astype(np.int32), c=g.integers(-3, 4, n).astype(np.int64))


def _run(P, q, p, x0, parts):
    ctx = P.qubo_gda_init(q, p, x0)
    for k in parts:
        ctx.step(k)
    x, y, t = ctx.get_state()
    r, F, tr, name = ctx.result(), ctx.objectives(), ctx.trace(), ctx.tile_name
    ctx.destroy()
    return dict(x=x, y=y, t=t, F=F, best_x=r["best_x"], obj=r["best_obj"], b=r["best_restart"],
                it=r["best_iter"], trt=tr["t"], trF=tr["F"], trb=tr["b"]), name


def _same(a, b, trace=True):
    for k in a:
        if trace or not k.startswith("tr"):
            assert np.array_equal(a[k], b[k]), k


# (n, degree, largest weight, hub, kappa even): one to sixteen rows per thread,
# both sides of each step; rows longer than the register-held groups
SIZES = [(1, 0, 1, 0, False), (63, 3, 1, 0, True), (65, 9, 1024, 0, False), (1024, 6, 1, 0, True),
         (1025, 5, 40, 200, False), (2049, 6, 1, 0, True), (4096, 7, 3, 0, False), (4097, 3, 1, 500, True),
         (8193, 4, 1, 0, False), (16384, 2, 7, 0, True)]


@pytest.mark.parametrize("n,deg,wmax,hub,even", SIZES)
def test_few_restarts_match_row_parallel(n, deg, wmax, hub, even):
    P = require_gpu()
    q = _graph(n, deg, 1, wmax, hub, even)
    B = 5
    x0 = W.x0_uniform(9, 1, B, n)
    x0[:, ::11] = 0.5
    for g in ("quad", "entropy"):
        say(f"[resident seq] n={n} deg={deg} wmax={wmax} hub={hub} g={g}")
        p = W.gda_params("qubo", B=B, T=1, scale=float(max(1, wmax)), g=g)
        a, name = _run(P, q, p, x0, [1, 2, 60])
        b, rows = _run(P, q, dict(p, tile=2), x0, [63])
        assert name == "csr_resident_seq" and rows == "csr_rows"
        _same(a, b)
        assert np.array_equal(a["F"], oq.objective(q, a["x"] > 0.5))


@pytest.mark.parametrize("n,deg,wmax,hub,even", SIZES)
def test_many_restarts_match_csr_order(n, deg, wmax, hub, even, monkeypatch):
    P = require_gpu()
    q = _graph(n, deg, 2, wmax, hub, even)
    B = 128
    x0 = W.x0_uniform(9, 2, B, n)
    say(f"[resident] n={n} deg={deg} wmax={wmax} hub={hub}")
    p = W.gda_params("qubo", B=B, T=1, scale=float(max(1, wmax)))
    a, _ = _run(P, q, p, x0, [3, 1, 36])
    monkeypatch.setenv("PDBO_CSR_SLICED", "0")
    b, _ = _run(P, q, p, x0, [40])
    _same(a, b)


def test_long_call_set_state_and_restart():
    """A call longer than one launch's records (1023 iterations), a state set
    in the middle with a count >= 1 (which is offered too) and a restart."""
    P = require_gpu()
    q = W.maxcut_c2(3, n=300, M=900)
    B = 7
    x0 = W.x0_uniform(9, 3, B, q.n)
    g = np.random.default_rng(5)
    X, Y = g.random((B, q.n)).astype(np.float32), g.uniform(-2, 6, (B, q.n)).astype(np.float32)
    out = []
    for tile in (0, 2):
        say(f"[resident seq] long call, tile={tile}")
        ctx = P.qubo_gda_init(q, W.gda_params("maxcut", B=B, T=1, tile=tile), x0)
        got = []
        for k in range(2):
            ctx.step(2100)
            ctx.set_state(X, Y, 2100)
            ctx.step(300)
            r, tr = ctx.result(), ctx.trace()
            got += [ctx.get_state(), ctx.objectives(), (r["best_obj"], r["best_iter"], r["best_restart"]),
                    r["best_x"], tr["t"], tr["F"], tr["b"]]
            ctx.restart(x0)
        ctx.destroy()
        out.append(got)
    for a, b in zip(*out):
        for u, v in zip(a, b) if isinstance(a, tuple) else [(a, b)]:
            assert np.array_equal(u, v)


@pytest.mark.parametrize("n,deg,wmax,B,auto,forced", [
    (300, 6, 1, 128, "csr_resident", "csr_packed_dbuf_t32"), (2000, 6, 3, 128, "csr_resident", "csr_sliced_dbuf_t32"),
    (2000, 60, 1, 130, "csr_resident", "csr_l2_dbuf_t32"), (2000, 6, 3, 300, "csr_sliced_dbuf_t32", "csr_sliced_dbuf_t32"),
    (2000, 6, 2049, 128, "csr_sliced_dbuf_t32", "csr_sliced_dbuf_t32")])
def test_name_tells_the_kernel(n, deg, wmax, B, auto, forced):
    """The automatic choice may take csr_resident, a caller who names the
    restart-resident path gets csr_persistent (whose variants for quadratic g and
    int32 totals keep a test that way); the name tells which, the bits do not."""
    P = require_gpu()
    q = _graph(n, deg, 4, wmax)
    x0 = W.x0_uniform(9, 4, B, n)
    say(f"[resident name] n={n} deg={deg} wmax={wmax} B={B}")
    p = W.gda_params("qubo", B=B, T=1, scale=float(wmax))
    a, name = _run(P, q, p, x0, [40])
    b, named = _run(P, q, dict(p, tile=1), x0, [1, 39])
    assert (name, named) == (auto, forced)
    _same(a, b)
    assert np.array_equal(a["F"], oq.objective(q, a["x"] > 0.5))


@pytest.mark.parametrize("n,deg,B,g,name", [
    (5000, 3, 128, "quad", "csr_sliced_dbuf_t32"), (7000, 3, 130, "quad", "csr_sliced_inplace_i32"),
    (4000, 4, 128, "quad", "csr_resident"), (9000, 1, 128, "entropy", "csr_resident"),
    (8000, 3, 128, "entropy", "csr_resident"), (2000, 6, 128, "entropy", "csr_sliced_dbuf_t32"),
    (4000, 40, 10, "quad", "csr_rows"), (2000, 60, 10, "quad", "csr_resident_seq"),
    (2000, 60, 10, "entropy", "csr_rows"), (12000, 3, 10, "entropy", "csr_rows"),
    (12000, 3, 10, "quad", "csr_resident_seq"), (12000, 3, 100, "entropy", "csr_resident_seq")])
def test_automatic_choice(n, deg, B, g, name, monkeypatch):
    """What the measured times choose, on both sides of each line."""
    P = require_gpu()
    monkeypatch.setenv("PDBO_ROUTE", "0")
    q = W.maxcut_c2(2, n=n, M=n * deg // 2)
    say(f"[resident choice] n={n} deg={deg} B={B} g={g}")
    ctx = P.qubo_gda_init(q, W.gda_params("maxcut", B=B, T=1, g=g), None)
    got = ctx.tile_name
    ctx.destroy()
    assert got == name


@pytest.mark.parametrize("n,deg,wmax,hub,even", SIZES)
def test_forced_resident_matches_persistent(n, deg, wmax, hub, even, monkeypatch):
    """csr_resident in csr_persistent's order wherever it can run, staged or
    streamed, with either g."""
    P = require_gpu()
    q = _graph(n, deg, 6, wmax, hub, even)
    B = 130
    x0 = W.x0_uniform(9, 6, B, n)
    x0[:, ::11] = 0.5
    for g in ("quad", "entropy"):
        say(f"[resident forced] n={n} deg={deg} wmax={wmax} hub={hub} g={g}")
        p = W.gda_params("qubo", B=B, T=1, scale=float(max(1, wmax)), g=g)
        out = []
        for force in ("1", "0"):
            monkeypatch.setenv("PDBO_CSR_RESIDENT", force)
            out.append(_run(P, q, p, x0, [2, 38]))
        assert out[0][1] == "csr_resident" and not out[1][1].startswith("csr_resident")
        _same(out[0][0], out[1][0])
