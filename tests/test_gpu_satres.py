"""The Max-k-SAT kernels on literals (k = 2..5, one workgroup per restart)
against the general kernels they stand in for (PDBO_SAT_RESIDENT=0): the same
sums in the same order and whole objectives, so runs, gradients and the
Lagrangian with its adjoint are compared bit for bit."""
import numpy as np
import pytest

import workloads as W
from gpu_util import require_gpu, say
from oracle import maxsat as om

pytestmark = pytest.mark.gpu

# (n, clauses per variable, k, largest weight): one to twenty positions per
# thread, both sides of each step and of the table's copies, lists of every
# length mod 4, the last size that fits and the first that does not, weights at
# and past what float16 holds exactly, and a formula in which more variables
# change in an iteration than the list in LDS takes (alpha 0.5)
CASES = [(5, 2.0, 3, 9, 0.01), (64, 4.2, 3, 2048, 0.01), (65, 3.1, 2, 5, 0.01), (1025, 9.0, 4, 10, 0.01),
         (2049, 4.2, 3, 10, 0.01), (4097, 5.3, 5, 7, 0.01), (5050, 4.2, 3, 2049, 0.01), (8193, 4.2, 3, 10, 0.5),
         (10060, 4.0, 4, 3, 0.01), (20266, 1.3, 3, 10, 0.01), (20267, 1.3, 3, 10, 0.01), (300, 2.0, 6, 4, 0.01)]


def _formula(n, ratio, k, wmax):
    f = W.random_maxsat(n, max(1, int(n * ratio)), k, 0, wmax, np.random.default_rng([n, k, wmax]))
    return f


@pytest.mark.parametrize("n,ratio,k,wmax,alpha", CASES)
def test_runs_match_general_kernels(n, ratio, k, wmax, alpha, monkeypatch):
    P = require_gpu()
    f = _formula(n, ratio, k, wmax)
    B = 3
    x0 = W.x0_uniform(5, 7, B, n)
    x0[:, ::9], x0[:, 1::11], x0[:, 2::13] = 0.5, 0.0, 1.0
    for g in ("entropy", "quad"):
        say(f"[satres] n={n} m={f.m} k={k} wmax={wmax} alpha={alpha} g={g}")
        p = W.gda_params("maxsat", B=B, T=1, scale=max(1.0, wmax / 2.0), g=g, alpha=alpha)
        out = []
        for res, parts in (("1", [1, 2, 30]), ("0", [33])):
            monkeypatch.setenv("PDBO_SAT_RESIDENT", res)
            ctx = P.maxsat_gda_init(f, p, x0)
            G = ctx.grad(x0.astype(np.float32))
            for t in parts:
                ctx.step(t)
            x, y, t = ctx.get_state()
            r = ctx.result()
            out.append((G, x, y, ctx.objectives(), r["best_x"], r["best_obj"], r["best_iter"], r["best_restart"]))
            ctx.destroy()
        for a, b in zip(*out):
            assert np.array_equal(a, b)
        assert np.array_equal(out[0][3], om.objective(f, out[0][1] > 0.5))
        assert out[0][5] == om.objective(f, out[0][4][None].astype(bool))[0]


@pytest.mark.parametrize("n,ratio,k,wmax,alpha", CASES[::2] + CASES[-3:-2])
def test_lagrangian_matches_general_kernels(n, ratio, k, wmax, alpha, monkeypatch):
    import torch
    P = require_gpu()
    f = _formula(n, ratio, k, wmax)
    nb = 2
    g = np.random.default_rng(3)
    x0 = g.random((nb, n))
    x0[:, ::9], x0[:, 1::11], x0[:, 2::13], x0[:, 3::17] = 0.5, 0.0, 1.0, 2.0 ** -22
    x = torch.from_numpy(x0.astype(np.float32)).cuda()
    y = torch.from_numpy(g.uniform(-1, 2, (nb, n)).astype(np.float32)).cuda()
    w = torch.tensor([0.75, -2.0], device="cuda")
    for kind in ("entropy", "quad"):
        say(f"[satres lagrangian] n={n} k={k} g={kind}")
        out = []
        for res in ("1", "0"):
            monkeypatch.setenv("PDBO_SAT_RESIDENT", res)
            ctx = P.maxsat_gda_init(f, W.gda_params("maxsat", B=1, T=1, scale=2.0, g=kind), None)
            L = P.maxsat_lagrangian_fwd(ctx, x, y)
            out.append((L, *P.maxsat_lagrangian_bwd(ctx, x, y, w)))
            torch.cuda.synchronize()
            ctx.destroy()
        for a, b in zip(*out):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n,m,k,wmax", [(64, 270, 3, 9), (65, 140, 2, 5), (1025, 4000, 4, 10), (2049, 8000, 3, 10),
                                        (4097, 20000, 5, 7), (16385, 30000, 3, 10)])
def test_lagrangian_outside_the_box_matches_general_kernels(n, m, k, wmax, monkeypatch):
    """x outside [0, 1] (the step of an optimizer that clamps afterwards), clauses
    of weight zero, and an x with NaN and infinities, which reach the variables
    that share a clause with them and no others."""
    import torch
    P = require_gpu()
    f = W.random_maxsat(n, m, k, 0, wmax, np.random.default_rng([n, k]))
    f.w[::7] = 0
    nb = 3
    g = np.random.default_rng(4)
    x0 = g.uniform(-0.2, 1.2, (nb, n)).astype(np.float32)
    x0[:, ::9], x0[:, 1::11], x0[:, 2::13] = 0.0, 1.0, np.nextafter(np.float32(1), np.float32(2))
    x0[2, 3], x0[2, 5], x0[2, n - 1] = np.nan, np.inf, -np.inf
    y0 = g.uniform(-1, 2, (nb, n)).astype(np.float32)
    x, y = torch.from_numpy(x0).cuda(), torch.from_numpy(y0).cuda()
    w = torch.tensor([0.75, -2.0, 1.0], device="cuda")
    for kind in ("entropy", "quad"):
        say(f"[satres outside] n={n} k={k} g={kind}")
        out = []
        for res in ("1", "0"):
            monkeypatch.setenv("PDBO_SAT_RESIDENT", res)
            ctx = P.maxsat_gda_init(f, W.gda_params("maxsat", B=1, T=1, scale=2.0, g=kind), None)
            L = P.maxsat_lagrangian_fwd(ctx, x, y)
            out.append([v.cpu().numpy() for v in (L, *P.maxsat_lagrangian_bwd(ctx, x, y, w))])
            ctx.destroy()
        for a, b in zip(*out):
            assert np.array_equal(a, b, equal_nan=True)
        assert np.isfinite(out[0][1][:2]).all() and 0 < np.isfinite(out[0][1][2]).sum() < n
        if kind == "quad":
            # the multilinear extension in float64: at most 1.2^(k-1) per factor
            # product, k + occurrences roundings of 2^-24 each
            X = torch.from_numpy(x0[:2].astype(np.float64)).requires_grad_()
            Y = torch.from_numpy(y0[:2].astype(np.float64))
            v, neg = torch.from_numpy(np.abs(f.lits) - 1).long(), torch.from_numpy(f.lits < 0)
            fac = torch.where(neg, X[:, v], 1 - X[:, v]).prod(-1)
            val = (fac * torch.from_numpy(f.w.astype(np.float64))).sum(-1) / 2.0 + (Y * (X * X - X)).sum(-1)
            (val * torch.tensor([0.75, -2.0], dtype=torch.float64)).sum().backward()
            occ = np.bincount(np.abs(f.lits).ravel() - 1, minlength=n).max()
            tol = 2.0 * (occ * wmax * 1.2 ** (k - 1) / 2.0 + 3.0) * (occ + k + 4) * 2.0 ** -24
            assert np.abs(out[0][1][:2] - X.grad.numpy()).max() <= tol


def test_no_room_for_the_layout(monkeypatch):
    """Without room for the layout on literals a formula runs on the general
    kernels, with the same bits."""
    P = require_gpu()
    f = _formula(700, 4.2, 3, 10)
    p = W.gda_params("maxsat", B=3, T=1, scale=5.0, seed=2)

    def run():
        ctx = P.maxsat_gda_init(f, p, None)
        ctx.step(40)
        out = [*ctx.get_state(), ctx.objectives(), ctx.result()["best_x"]]
        ctx.destroy()
        return out

    monkeypatch.setenv("PDBO_SAT_RESIDENT", "0")
    ref = run()
    monkeypatch.setenv("PDBO_SAT_RESIDENT", "1")
    refused = []
    for k in range(1, 25):
        say(f"[satres enomem] allocation {k}")
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", str(k))
        try:
            for a, b in zip(run(), ref):
                assert np.array_equal(a, b)
        except P.PdboError as e:
            assert e.status == 2
            refused.append(k)
        monkeypatch.setenv("PDBO_FAIL_ALLOC_AT", "0")
    last = max(refused)
    assert len(refused) == last - 1  # one of them is the layout's
