"""Max-k-Cut with one workgroup per restart against the row-parallel kernels it
stands in for (PDBO_KCUT_RESIDENT=0): the same operations in the same order, so
runs, incumbents and traces are compared bit for bit."""
import numpy as np
import pytest

import workloads as W
from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

# (n, edges, k, g, y0): every k, one to sixteen positions per thread, one, two
# and four copies of X, isolated nodes, long rows; the last ones run into more
# changed nodes in an iteration than the list in LDS takes (alpha 0.9)
CASES = [(1, 0, 2, "quad", 0.01), (63, 100, 3, "entropy", 0.01), (65, 2000, 8, "quad", 0.01),
         (1025, 900, 6, "entropy", 0.01), (2049, 9000, 7, "quad", 0.01), (3000, 4000, 4, "entropy", 0.01),
         (4096, 9000, 8, "quad", 0.01), (6000, 12000, 5, "quad", 0.01), (10240, 20000, 3, "entropy", 0.01),
         (16384, 16000, 2, "quad", 0.01), (9000, 60000, 3, "quad", 0.9), (16385, 16000, 2, "quad", 0.01)]


def _params(B, g, alpha, **over):
    return dict(dict(B=B, T=1, alpha=alpha, beta=0.01, y0=0.5, delta=2.0 ** -7, scale=1.0, g=g, seed=3), **over)


@pytest.mark.parametrize("n,m,k,kind,alpha", CASES)
def test_runs_match_row_parallel(n, m, k, kind, alpha, monkeypatch):
    P = require_gpu()
    g = W.kcut_graph(n, m, k, rep=4) if m else W.Kcut(n=n, k=k, row_ptr=np.zeros(n + 1, np.int32),
                                                      col_idx=np.zeros(0, np.int32), w=np.zeros(0, np.int32))
    if n == 65:
        g.w = (g.w * 2048).astype(np.int32)
    out = []
    for res, parts in (("1", [1, 2, 30]), ("0", [33])):
        say(f"[kcut resident] n={n} m={m} k={k} g={kind} resident={res}")
        monkeypatch.setenv("PDBO_KCUT_RESIDENT", res)
        ctx = P.kcut_gda_init(g, _params(4, kind, alpha), None)
        for t in parts:
            ctx.step(t)
        Z, Y, t = ctx.get_state()
        r, tr = ctx.result(), ctx.trace()
        out.append((Z, Y, t, ctx.objectives(), r["best_obj"], r["best_iter"], r["best_restart"], r["best_x"],
                    tr["t"], tr["F"], tr["b"], ctx.grad(Z), ctx.eval(np.tile(r["best_x"], (2, 1)))))
        ctx.destroy()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert out[0][4] == out[0][-1][0]


def test_long_call_set_state_and_restart(monkeypatch):
    """A call longer than one launch's records, a state set in the middle with a
    count >= 1 (which is offered too), logits alone and duals alone, a restart."""
    P = require_gpu()
    g = W.kcut_graph(300, 900, 3, rep=6)
    B = 5
    rng = np.random.default_rng(1)
    Z, Y = rng.normal(size=(B, 300, 3)).astype(np.float32), rng.normal(size=(B, 300)).astype(np.float32)
    out = []
    for res in ("1", "0"):
        monkeypatch.setenv("PDBO_KCUT_RESIDENT", res)
        ctx = P.kcut_gda_init(g, _params(B, "quad", 0.05), None)
        got = []
        for x, y in ((Z, Y), (Z, None), (None, Y)):
            say(f"[kcut resident] long call, resident={res}")
            ctx.step(1100)
            ctx.set_state(x, y, 1100)
            ctx.step(50)
            r, tr = ctx.result(), ctx.trace()
            got += [*ctx.get_state(), ctx.objectives(), r["best_obj"], r["best_iter"], r["best_restart"],
                    r["best_x"], tr["t"], tr["F"], tr["b"]]
            ctx.restart(None)
        ctx.destroy()
        out.append(got)
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("B", [7, 600])
def test_times_of_improvements(B, monkeypatch):
    """More restarts than run at once: the improvements' times do not fall as t
    grows, the result's is the last one's, and the records are the row-parallel
    kernels'."""
    P = require_gpu()
    g = W.kcut_graph(2000, 4000, 3, rep=7)
    out = []
    for res in ("1", "0"):
        say(f"[kcut times] B={B} resident={res}")
        monkeypatch.setenv("PDBO_KCUT_RESIDENT", res)
        ctx = P.kcut_gda_init(g, _params(B, "quad", 0.01), None)
        for t in (150, 50, 300):
            ctx.step(t)
        tr, r = ctx.trace(), ctx.result()
        ctx.destroy()
        assert len(tr["t"]) > 20 and (np.diff(tr["t"]) > 0).all()
        assert (np.diff(tr["sec"]) >= 0).all() and tr["sec"][0] >= 0 and r["time_to_best_s"] == tr["sec"][-1]
        out.append((tr["t"], tr["F"], tr["b"], r["best_obj"], r["best_x"]))
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n,m,k", [(300, 450, 2), (2000, 3000, 3), (3000, 8000, 4), (1500, 2000, 7)])
def test_nan_stays_with_its_neighbours(n, m, k, monkeypatch):
    """A dual so large that the logits of its node overflow: NaN reaches the node's
    neighbours, an edge at an iteration, and no other node; an edge of weight zero
    carries it too."""
    P = require_gpu()
    g = W.kcut_graph(n, m, k, rep=8)
    hub = int(np.diff(g.row_ptr).argmax())
    far = int(g.col_idx[g.row_ptr[hub]])
    for i, j in ((hub, far), (far, hub)):
        g.w[g.row_ptr[i] + int(np.searchsorted(g.col_idx[g.row_ptr[i]:g.row_ptr[i + 1]], j))] = 0
    B = 4
    Y = np.full((B, n), 0.5, np.float32)
    Y[1, hub] = Y[2, n // 2] = 3e38
    for kind in ("quad", "entropy"):
        out = []
        for res in ("1", "0"):
            say(f"[kcut nan] n={n} k={k} g={kind} resident={res}")
            monkeypatch.setenv("PDBO_KCUT_RESIDENT", res)
            ctx = P.kcut_gda_init(g, _params(B, kind, 0.01), None)
            ctx.set_state(None, Y, 0)
            got = []
            for t in (1, 1, 2):
                ctx.step(t)
                got += [*ctx.get_state()[:2], ctx.objectives()]
            r, tr = ctx.result(), ctx.trace()
            got += [r["best_obj"], r["best_x"], tr["t"], tr["F"], tr["b"]]
            ctx.destroy()
            out.append(got)
        for a, b in zip(*out):
            a, b = np.asarray(a), np.asarray(b)
            assert np.array_equal(a, b, equal_nan=a.dtype == np.float32)
        if kind == "quad":
            # 2 x y overflows at the first or, x being a unit vector by then, the
            # second iteration; after four NaN is one to three edges away
            bad = np.isnan(out[1][6].reshape(B, n, k)).any(axis=2)
            near = np.zeros(n, bool)
            near[hub] = True
            row = np.repeat(np.arange(n), np.diff(g.row_ptr))
            for _ in range(3):
                near[g.col_idx[near[row]]] = True
            assert not bad[0].any() and bad[1, hub] and bad[1, far] and (bad[1] <= near).all()
