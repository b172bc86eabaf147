"""Few restarts with a restart's x in LDS range by range (PDBO_CSR_SPLIT=1)
against the row-parallel kernel it stands in for (0): the same sums in the same
order, so runs, incumbents and traces are compared bit for bit."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W
from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


def _graph(n, m, wmax, seed):
    """A random upper triangle with about m entries, row 0 long, linear terms."""
    rng = np.random.default_rng(seed)
    i, j = rng.integers(0, n, m), rng.integers(0, n, m)
    i[: m // 20] = 0
    keep = i < j
    M = sp.csr_matrix((np.ones(keep.sum()), (i[keep], j[keep])), shape=(n, n))
    M.sum_duplicates()
    w = rng.integers(-wmax, wmax + 1, M.nnz).astype(np.int32)
    if M.nnz:
        w[0] = wmax
    return W.Qubo(n=n, row_ptr=M.indptr.astype(np.int32), col_idx=M.indices.astype(np.int32), vals=w,
                  c=rng.integers(-50, 51, n).astype(np.int64))


# one range and the first size with two, slices of 64 rows, one to eight slices
# a wave, one restart to 64, the largest exact weight
CASES = [(1, 0, 1, 1, "quad"), (63, 300, 5, 3, "quad"), (130, 900, 2048, 64, "entropy"),
         (5000, 20000, 7, 10, "quad"), (40000, 100000, 3, 2, "entropy"), (40001, 100000, 3, 5, "quad"),
         (50000, 400000, 9, 64, "quad"), (65536, 90000, 4, 3, "poly")]


@pytest.mark.parametrize("n,m,wmax,B,g", CASES)
def test_matches_row_parallel(n, m, wmax, B, g, monkeypatch):
    P = require_gpu()
    q = _graph(n, m, wmax, n)
    rng = np.random.default_rng(1)
    x, y = rng.random((B, n)).astype(np.float32), rng.normal(size=(B, n)).astype(np.float32)
    out = []
    for split, chunk in (("0", 0), ("1", 0), ("1", 4)):
        say(f"[rowsplit] n={n} m={m} B={B} g={g} split={split} graph={chunk}")
        monkeypatch.setenv("PDBO_CSR_SPLIT", split)
        par = W.gda_params("qubo", B=B, T=1, scale=3.0, tile=2, g=g, g_degree=2, graph_chunk=chunk, seed=9)
        ctx = P.qubo_gda_init(q, par, None)
        assert ctx.tile_name == ("csr_split" if split == "1" else "csr_rows")
        got = []
        for sx, sy in ((None, None), (x, y), (None, y)):
            if sy is not None:
                ctx.set_state(sx, sy, 2)
            ctx.step(9)
            ctx.step(1)
            r, tr = ctx.result(), ctx.trace()
            got += [*ctx.get_state(), ctx.objectives(), r["best_obj"], r["best_iter"], r["best_restart"],
                    r["best_x"], tr["t"], tr["F"], tr["b"], ctx.grad(x), ctx.eval(r["best_x"][None])]
        ctx.restart(x.astype(np.float64))
        ctx.step(3)
        got += [*ctx.get_state(), ctx.objectives()]
        if g == "quad":
            d = P.qubo_dual_bound(ctx, 5)
            got += [d[k] for k in sorted(d)]
        ctx.destroy()
        out.append(got)
    for got in out[1:]:
        for k, (a, b) in enumerate(zip(got, out[0])):
            assert np.array_equal(a, b), k


def test_wider_weights_stay_row_parallel(monkeypatch):
    P = require_gpu()
    monkeypatch.setenv("PDBO_CSR_SPLIT", "1")
    ctx = P.qubo_gda_init(_graph(300, 2000, 2049, 4),
                          W.gda_params("qubo", B=4, T=1, scale=3.0, tile=2), None)
    assert ctx.tile_name == "csr_rows"
    ctx.destroy()
