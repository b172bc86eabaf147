"""Step launches with one wave a tile (operands in fragment order) against the
workgroup tiles whose K order they keep (PDBO_FRAG=0): the same products added
in the same order, so runs are compared bit for bit."""
import numpy as np
import pytest

import workloads as W
from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

# n around the 16-row groups, one chunk up to more than two rounds of the eight
# in flight, B around the 16- and 32-column tiles; both K orders of the
# workgroup tiles occur (asserted in test_both_orders)
SIZES = [(1, 1), (16, 17), (129, 16), (700, 33), (1100, 5), (333, 100), (260, 700), (2100, 40)]
PRECS = ["fp32", "bf16", "fp8", "i8"]


def _choose(P, q, B, prec, g, cfg, path, monkeypatch):
    """Makes the tile configuration of this shape `cfg`: 1 a register-staged
    tile, 9 a direct-to-LDS one (their K orders differ)."""
    monkeypatch.setenv("PDBO_AUTOTUNE", "1")
    monkeypatch.setenv("PDBO_AUTOTUNE_CACHE", str(path))
    key = "gfx950/p%d/g%d/B%d/k1/nmax%d/nsum%d" % (P._PREC[prec], P._G[g], B, (q.n + 63) // 64 * 64,
                                                   (q.n + 1023) // 1024 * 1024)
    assert P.load().pdbo_autotune_store(key.encode(), cfg) == 0


def _run(P, q, B, prec, g, frag, monkeypatch, eval_every=1):
    monkeypatch.setenv("PDBO_FRAG", frag)
    par = W.gda_params("qubo", B=B, T=1, scale=40.0 * q.n ** 0.5, precision=prec, g=g, eval_every=eval_every)
    ctx = P.qubo_gda_init(q, par, None)
    name = ctx.tile_name
    rng = np.random.default_rng(q.n)
    x, y = rng.random((B, q.n)).astype(np.float32), rng.normal(size=(B, q.n)).astype(np.float32)
    got = []
    for sx, sy in ((None, None), (x, y), (None, y), (x, None)):
        if sx is not None or sy is not None:
            ctx.set_state(sx, sy, 3)
        ctx.step(3)
        ctx.step(2)
        X, Y, t = ctx.get_state()
        r, tr = ctx.result(), ctx.trace()
        got += [X, Y, t, ctx.objectives(), r["best_obj"], r["best_iter"], r["best_restart"], r["best_x"],
                tr["F"], ctx.grad(x)]
    ctx.restart(x.astype(np.float64))
    ctx.step(4)
    got += [*ctx.get_state(), ctx.objectives()]
    if g == "quad":
        d = P.qubo_dual_bound(ctx, 9)
        got += [d[k] for k in sorted(d)] if isinstance(d, dict) else list(d)
    ctx.destroy()
    return name, got


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n,B", SIZES)
@pytest.mark.parametrize("cfg,g", [(1, "quad"), (9, "quad"), (9, "entropy")])
def test_matches_workgroup_tiles(n, B, prec, cfg, g, monkeypatch, tmp_path):
    P = require_gpu()
    q = W.random_dense_qubo(n, -100, 100, W.rng_for(3, 0, 0, n))
    if prec == "i8":
        q = W.random_dense_qubo(n, -60, 60, W.rng_for(3, 0, 0, n))
    say(f"[frag] n={n} B={B} prec={prec} g={g} tile={cfg}")
    _choose(P, q, B, prec, g, cfg, tmp_path / "tiles.json", monkeypatch)
    name, want = _run(P, q, B, prec, g, "0", monkeypatch)
    assert name == {1: "64x64_w2x2_0", 9: "64x64_w2x2_1"}[cfg]
    for frag in ("1", "2"):
        name, got = _run(P, q, B, prec, g, frag, monkeypatch)
        assert name == "frag_16x16x" + frag
        for k, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b), (frag, k)


@pytest.mark.parametrize("grouped", [True, False])
def test_batches_and_graphs(grouped, monkeypatch):
    """Uneven instances in one context, recorded iterations, full products only."""
    P = require_gpu()
    qs = [W.random_dense_qubo(n, -60, 60, W.rng_for(4, 0, 0, n)) for n in (40, 333, 129)]
    out = []
    for frag in ("0", "1", "2"):
        say(f"[frag] batch grouped={grouped} frag={frag}")
        monkeypatch.setenv("PDBO_FRAG", frag)
        monkeypatch.setenv("PDBO_AUTOTUNE", "0")
        ps = [W.gda_params("qubo", B=20, T=1, scale=40.0 * q.n ** 0.5, precision="i8", graph_chunk=8, seed=5)
              for q in qs]
        ctx = P.qubo_gda_batch_init(qs, ps, [None] * 3, grouped=grouped)
        ctx.step(100)
        ctx.step(30)
        got = []
        for i in range(3):
            r = P.qubo_gda_batch_result(ctx, i)
            got += [r["best_obj"], r["best_iter"], r["best_restart"], r["best_x"]]
        ctx.destroy()
        out.append(got)
    for got in out[1:]:
        for a, b in zip(got, out[0]):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("tile", [2, 10])
def test_dual_of_tiled_contexts(tile, prec, monkeypatch):
    """A context on workgroup tiles takes its certificate's descent by one-wave tiles."""
    P = require_gpu()
    q = W.random_dense_qubo(500, -60, 60, W.rng_for(5, 0, 0, 500))
    out = []
    for frag in ("0", None):
        say(f"[frag] dual tile={tile} prec={prec} frag={frag}")
        if frag is None:
            monkeypatch.delenv("PDBO_FRAG", raising=False)
        else:
            monkeypatch.setenv("PDBO_FRAG", frag)
        par = W.gda_params("qubo", B=70, T=1, scale=40.0 * 500 ** 0.5, precision=prec, tile=tile, seed=2)
        ctx = P.qubo_gda_init(q, par, None)
        ctx.step(3)
        d = [P.qubo_dual_bound(ctx, 20) for _ in range(2)]
        ctx.step(3)
        out.append([e[k] for e in d for k in sorted(e)] + [ctx.objectives(), *ctx.get_state()])
        ctx.destroy()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_no_room_for_the_copies(monkeypatch):
    """The operands in fragment order are optional: an allocation of theirs that
    fails leaves the context on its tiles, with the same run, and frees the rest."""
    import torch
    P = require_gpu()
    q = W.random_dense_qubo(900, -60, 60, W.rng_for(5, 1, 0, 900))
    par = W.gda_params("qubo", B=20, T=1, scale=600.0, precision="i8", seed=3)

    def run():
        ctx = P.qubo_gda_init(q, par, None)
        name = ctx.tile_name
        ctx.step(70)
        out = [ctx.objectives(), *ctx.get_state(), ctx.result()["best_x"]]
        ctx.destroy()
        return name, out

    ref_name, ref = run()
    assert ref_name.startswith("frag")
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    refused = fell_back = 0
    for k in range(1, 40):
        say(f"[frag enomem] allocation {k}")
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", str(k))
        try:
            name, got = run()
            fell_back += not name.startswith("frag")
            for a, b in zip(got, ref):
                assert np.array_equal(a, b)
        except P.PdboError as e:
            assert e.status == 2
            refused += 1
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", "0")
        assert torch.cuda.mem_get_info()[0] >= free0 - (2 << 20), k
    assert fell_back == 4 and refused >= 5  # A, the two shadows and the tile table
