"""Workloads for timing the library through its public entry points.

A case is a dict of plain values.  `prepare` makes what a user's program holds
before the call (the instance uploaded in a context, or device tensors), `run`
is one pass, `exact` the same outputs in float64 without this library, and
`work` the bytes and operations one pass cannot do without.

Kinds
  solve    restart on fresh starting points, T iterations of Alg. 1, and the
           incumbent with the objectives of every restart ("state": also the
           iterate, which a program reads for a checkpoint): a dense, CSR,
           MIS, Max-SAT or Max-k-Cut instance, by "family"
  batch    many dense instances of uneven size stepped together
  lagr     the smoothed Max-SAT Lagrangian forward and backward (autograd)
  dual     the dual certificate
  eval     exact objectives of device vectors without allocation
"""
import math

import numpy as np
import torch

import paper_2509_21064_amd as pdbo

DELTA = 2.0 ** -7
HYPER = {  # y0, alpha, beta by family
    "dense": (6.0, 0.025, 0.025),
    "csr": (6.0, 0.025, 0.025),
    "mis": (5.0, 0.02, 0.02),
    "sat": (2.0, 0.01, 0.005),
    "kcut": (6.0, 0.01, 0.01),
}


def listed():
    return [
        # the smallest call: a 200-node graph with +-1 weights given dense, a
        # handful of restarts; launches and latency are what counts
        dict(name="dense_fp32_n200_B16", kind="solve", family="dense", n=200, p=0.05, B=16, T=150, prec="fp32",
             g="quad", graph=0, state=True),
        # an ordinary dense QUBO, ragged size, the usual hundred restarts, bf16 operands
        dict(name="dense_bf16_n3001_B100", kind="solve", family="dense", n=3001, p=1.0, B=100, T=150, prec="bf16",
             g="quad", graph=0, state=True),
        # the headline workload: dense n = 10^4, 1024 restarts, int8 operands
        dict(name="dense_i8_n10000_B1024", kind="solve", family="dense", n=10000, p=1.0, B=1024, T=200, prec="i8",
             g="quad", graph=0, state=False),
        # Max-Cut on a sparse graph with the hundred restarts the method's hyper-parameters name
        dict(name="maxcut_n2000_B100", kind="solve", family="csr", n=2000, deg=6, B=100, T=1000, g="quad", graph=0,
             state=False),
        # the same graph with a restart for every compute unit
        dict(name="maxcut_n2000_B256", kind="solve", family="csr", n=2000, deg=6, B=256, T=5000, g="quad", graph=0,
             state=False),
        # maximum independent set on a large 100-regular graph, ten restarts, recorded iterations
        dict(name="mis_n50000_d100_B10", kind="solve", family="mis", n=50000, deg=100, B=10, T=400, g="quad",
             graph=50, state=True),
        # Max-3-Cut on a sparse graph, a hundred restarts, recorded iterations
        dict(name="max3cut_n10000_B100", kind="solve", family="kcut", n=10000, deg=4, k=3, B=100, T=200, g="quad",
             graph=50, state=False),
        # weighted random 3-SAT at the hard ratio
        dict(name="sat3_n20000_B256", kind="solve", family="sat", n=20000, ratio=4.2, k=3, B=256, T=100, g="entropy",
             graph=0, state=False),
        # weighted random 5-SAT: longer clauses, many occurrences per variable
        dict(name="sat5_n4000_B100", kind="solve", family="sat", n=4000, ratio=20.0, k=5, B=100, T=100, g="entropy",
             graph=0, state=True),
        # sixteen dense instances of uneven size in one context, recorded iterations
        dict(name="batch16_i8_B128", kind="batch", count=16, lo=500, hi=5000, B=128, T=200, prec="i8", graph=50),
        # a torch program differentiating the smoothed Max-SAT Lagrangian
        dict(name="lagrangian_n20000_B256", kind="lagr", n=20000, ratio=4.2, k=3, B=256, g="entropy"),
        # a certified lower bound for a dense instance
        dict(name="dual_i8_n5000", kind="dual", n=5000, B=16, iters=300, prec="i8"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(n):
    return n + (n & 1)


def draw(rng):
    kind = rng.choice(["dense", "dense", "csr", "csr", "mis", "kcut", "sat", "sat", "batch", "lagr", "dual", "eval"])
    if kind == "dense":
        n, B, prec = _log(rng, 60, 9000), _log(rng, 10, 1024), rng.choice(["fp32", "bf16", "i8", "fp8"])
        small = n <= 800 and rng.random() < 0.5
        # iterations so that a pass stays below the headline workload's
        rate = {"fp32": 0.6e14, "bf16": 4e14, "i8": 8e14, "fp8": 8e14}[prec]
        T = max(4, min(_log(rng, 20, 300), int(0.02 / (2.0 * n * n * B / rate + 2e-5))))
        return dict(kind="solve", family="dense", n=n, p=0.05 if small else 1.0, B=B, T=T, prec=prec,
                    g=rng.choice(["quad", "quad", "entropy"]), graph=0, state=n * B <= 1 << 19 and T <= 150)
    if kind == "csr":
        n, B = _log(rng, 200, 12000), _log(rng, 10, 400)
        T = min(_log(rng, 50, 1000), int(0.02 / (2e-5 + 2e-12 * n * 6 * B)))
        return dict(kind="solve", family="csr", n=n, deg=rng.choice([3, 4, 6, 12]), B=B, T=T,
                    g=rng.choice(["quad", "quad", "entropy"]), graph=rng.choice([0, 50]),
                    state=n * B <= 1 << 18 and T <= 150)
    if kind == "mis":
        n, d, B = _even(_log(rng, 1000, 50000)), rng.choice([3, 5, 20, 100]), rng.choice([1, 5, 10, 20, 48])
        if n * d * B > 60e6:
            B = 10
        return dict(kind="solve", family="mis", n=n, deg=d, B=B, T=_log(rng, 50, 200), g="quad",
                    graph=rng.choice([0, 50]), state=True)
    if kind == "kcut":
        n, k, B = _log(rng, 200, 10000), rng.choice([2, 3, 3, 4, 6]), _log(rng, 10, 128)
        T = min(_log(rng, 50, 200), int(0.02 / (3e-5 + 2e-11 * n * k * B)))
        return dict(kind="solve", family="kcut", n=n, deg=rng.choice([4, 8]), k=k, B=B, T=T,
                    g=rng.choice(["quad", "entropy"]), graph=rng.choice([0, 50]), state=False)
    if kind == "sat":
        k = rng.choice([2, 3, 3, 4, 5])
        ratio = {2: 2.0, 3: 4.2, 4: 9.0, 5: 20.0}[k]
        n = _log(rng, 300, {2: 24000, 3: 20000, 4: 8000, 5: 4000}[k])
        B, T = _log(rng, 10, 256), _log(rng, 20, 100)
        if k > 3:
            T = max(4, min(T, int(4e9 / (n * ratio * k * B))))
        return dict(kind="solve", family="sat", n=n, ratio=ratio, k=k, B=B, T=T,
                    g=rng.choice(["entropy", "entropy", "quad"]), graph=0, state=n * B <= 1 << 19)
    if kind == "batch":
        lo = _log(rng, 100, 800)
        return dict(kind="batch", count=rng.randint(3, 12), lo=lo, hi=rng.randint(lo + 200, 3500),
                    B=_log(rng, 16, 128), T=_log(rng, 70, 150), prec=rng.choice(["i8", "bf16"]),
                    graph=rng.choice([0, 50]))
    if kind == "lagr":
        return dict(kind="lagr", n=_log(rng, 300, 20000), ratio=4.2, k=rng.choice([3, 3, 3, 4]), B=_log(rng, 1, 256),
                    g="entropy")
    if kind == "dual":
        return dict(kind="dual", n=_log(rng, 300, 6000), B=16, iters=_log(rng, 50, 300), prec="i8")
    fam = rng.choice(["dense", "csr", "sat", "kcut"])
    c = dict(kind="eval", family=fam, B=_log(rng, 8, 512))
    if fam == "dense":
        c.update(n=_log(rng, 100, 4000), p=1.0)
    elif fam == "csr":
        c.update(n=_log(rng, 200, 20000), deg=rng.choice([6, 12]))
    elif fam == "sat":
        c.update(n=_log(rng, 300, 20000), k=3, ratio=4.2)
    else:
        c.update(n=_log(rng, 200, 10000), deg=4, k=3)
    return c


# ---------------------------------------------------------------- instances


class _Obj:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def _dense_qubo(case, seed):
    """p = 1: symmetric weights U{-100..100} with linear terms; p < 1: a
    G(n, p) graph with +-1 weights, c = 0."""
    n, gen = case["n"], torch.Generator(device="cuda").manual_seed(seed * 7919 + 1)
    if case.get("p", 1.0) >= 1.0:
        Q = torch.randint(-100, 101, (n, n), generator=gen, device="cuda", dtype=torch.int32)
        Q = torch.triu(Q) + torch.triu(Q, 1).T
        c = torch.randint(-100, 101, (n,), generator=gen, device="cuda", dtype=torch.int64)
        scale = max(1.0, 0.5 * math.sqrt(n * 3366.7))  # -lambda_min / 4 by the semicircle law
        return _Obj(n=n, Q=Q.cpu().numpy(), c=c.cpu().numpy()), scale
    keep = torch.rand((n, n), generator=gen, device="cuda") < case["p"]
    sign = torch.randint(0, 2, (n, n), generator=gen, device="cuda", dtype=torch.int32) * 2 - 1
    Q = torch.triu(sign * keep, 1).to(torch.int32)
    return _Obj(n=n, Q=(Q + Q.T).contiguous().cpu().numpy(), c=None), 1.0


def _edges(n, m, rng):
    """About m distinct edges i < j, uniform."""
    a, b = rng.integers(0, n, size=m + m // 8 + 16), rng.integers(0, n, size=m + m // 8 + 16)
    ok = a != b
    keys = np.unique(np.minimum(a, b)[ok].astype(np.int64) * n + np.maximum(a, b)[ok])
    if len(keys) > m:
        keys = np.sort(rng.permutation(keys)[:m])
    return keys // n, keys % n


def _csr(n, i, j, w):
    ii, jj, ww = np.concatenate([i, j]), np.concatenate([j, i]), np.concatenate([w, w]).astype(np.int32)
    order = np.argsort(ii.astype(np.int64) * n + jj)
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(ii, minlength=n), out=rp[1:])
    return rp.astype(np.int32), jj[order].astype(np.int32), ww[order]


def _maxcut(case, seed):
    """Max-Cut on G(n, n deg / 2) with +-1 weights: Q = W, c = -W 1."""
    n, rng = case["n"], np.random.default_rng([2, seed])
    i, j = _edges(n, n * case["deg"] // 2, rng)
    rp, col, val = _csr(n, i, j, np.where(rng.random(len(i)) < 0.5, 1, -1))
    c = -np.bincount(np.repeat(np.arange(n), np.diff(rp)), weights=val, minlength=n).astype(np.int64)
    return _Obj(n=n, Q=None, row_ptr=rp, col_idx=col, vals=val, c=c), 1.0


def _mis(case, seed):
    """-sum x_i + 4 sum_E x_i x_j on a random graph of degree d: a random
    pairing of the half-edges without its few loops and repeats."""
    n, d, rng = case["n"], case["deg"], np.random.default_rng([6, seed])
    s = rng.permutation(np.repeat(np.arange(n, dtype=np.int64), d))
    a, b = s[0::2], s[1::2]
    ok = a != b
    keys = np.unique(np.minimum(a, b)[ok] * n + np.maximum(a, b)[ok])
    rp, col, val = _csr(n, keys // n, keys % n, np.full(len(keys), 2))
    scale = max(1.0, math.sqrt(d - 1.0)) / (2.0 if d >= 50 else 1.0)
    return _Obj(n=n, Q=None, row_ptr=rp, col_idx=col, vals=val, c=np.full(n, -1, dtype=np.int64)), scale


def _kcut(case, seed):
    n, rng = case["n"], np.random.default_rng([7, seed])
    i, j = _edges(n, n * case["deg"] // 2, rng)
    rp, col, w = _csr(n, i, j, np.where(rng.random(len(i)) < 0.5, 1, -1))
    return _Obj(n=n, k=case["k"], row_ptr=rp, col_idx=col, w=w), 1.0


def _sat(case, seed):
    n, k, rng = case["n"], case["k"], np.random.default_rng([5, seed])
    m = int(n * case["ratio"])
    v = rng.integers(0, n, size=(m, k))
    while True:
        srt = np.sort(v, axis=1)
        bad = np.any(srt[:, 1:] == srt[:, :-1], axis=1)
        if not bad.any():
            break
        v[bad] = rng.integers(0, n, size=(int(bad.sum()), k))
    lits = np.where(rng.random((m, k)) < 0.5, -(v + 1), v + 1).astype(np.int32)
    w = rng.integers(1, 11, size=m).astype(np.int32)
    return _Obj(n=n, lits=lits, w=w), float(np.mean(w))


_MAKE = {"dense": _dense_qubo, "csr": _maxcut, "mis": _mis, "kcut": _kcut, "sat": _sat}


def _params(case, family, scale, seed):
    y0, alpha, beta = HYPER[family]
    return dict(B=case["B"], alpha=alpha, beta=beta, y0=y0, delta=DELTA, scale=scale, g=case.get("g", "quad"),
                precision=case.get("prec", "fp32"), graph_chunk=case.get("graph", 0), seed=seed)


def _context(case, family, seed):
    inst, scale = _MAKE[family](case, seed)
    init = {"sat": pdbo.maxsat_gda_init, "kcut": pdbo.kcut_gda_init}.get(family, pdbo.qubo_gda_init)
    return inst, scale, init(inst, _params(case, family, scale, seed), None)


def _batch_instances(case, seed):
    """Sizes U{lo..hi} and densities U[1%, 10%] (the same for every seed),
    weights U{-10..10}, c = 0."""
    shape, out, scales = np.random.default_rng([4, case["count"], case["lo"], case["hi"]]), [], []
    rng = np.random.default_rng([4, seed])
    for _ in range(case["count"]):
        n, rho = int(shape.integers(case["lo"], case["hi"] + 1)), float(shape.uniform(0.01, 0.10))
        i, j = _edges(n, max(1, int(rho * n * (n - 1) / 2)), rng)
        rp, col, val = _csr(n, i, j, rng.integers(-10, 11, size=len(i)))
        out.append(_Obj(n=n, Q=None, row_ptr=rp, col_idx=col, vals=val, c=None))
        scales.append(max(1.0, 0.5 * math.sqrt(n * rho * 36.67)))
    return out, scales


def _lagr_inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed * 104729 + 3)
    shape = (case["B"], case["n"])
    x = torch.rand(shape, generator=gen, device="cuda")
    y = 2.0 * torch.rand(shape, generator=gen, device="cuda") - 0.5
    w = torch.rand(case["B"], generator=gen, device="cuda") + 0.5
    return x, y, w


# ---------------------------------------------------------------- the passes


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        _, _, ctx = _context(case, case["family"], seed)
        return dict(case=case, ctx=ctx)
    if kind == "batch":
        qs, scales = _batch_instances(case, seed)
        ps = [_params(case, "dense", s, seed + 1000 * i) for i, s in enumerate(scales)]
        ctx = pdbo.qubo_gda_batch_init(qs, ps, [None] * len(qs))
        return dict(case=case, ctx=ctx)
    if kind == "lagr":
        inst, scale = _sat(case, seed)
        ctx = pdbo.maxsat_gda_init(inst, _params(dict(case, B=1), "sat", scale, seed), None)
        x, y, w = _lagr_inputs(case, seed)
        return dict(case=case, ctx=ctx, x=x.requires_grad_(), y=y.requires_grad_(), w=w)
    if kind == "dual":
        inst, scale = _dense_qubo(case, seed)
        return dict(case=case, ctx=pdbo.qubo_gda_init(inst, _params(case, "dense", scale, seed), None))
    _, _, ctx = _context(case, case["family"], seed)
    gen = torch.Generator(device="cuda").manual_seed(seed * 15485863 + 5)
    top = case["k"] if case["family"] == "kcut" else 2
    xr = torch.randint(0, top, (case["B"], case["n"]), generator=gen, device="cuda", dtype=torch.uint8)
    return dict(case=case, ctx=ctx, xr=xr, F=torch.zeros(case["B"], device="cuda", dtype=torch.int64))


def _found(r):
    return dict(best_obj=r["best_obj"], best_restart=r["best_restart"], best_iter=r["best_iter"],
                best_x=r["best_x"])


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "solve":
        ctx.restart(None)
        ctx.step(case["T"])
        out = _found(ctx.result())
        out["F"] = ctx.objectives()
        if case["state"]:
            out["x"], out["y"], _ = ctx.get_state()
        return out
    if kind == "batch":
        # a batched context has no restart: each pass goes on from the last one
        ctx.step(case["T"])
        rs = [pdbo.qubo_gda_batch_result(ctx, i) for i in range(case["count"])]
        return dict(best_obj=np.array([r["best_obj"] for r in rs]),
                    best_iter=np.array([r["best_iter"] for r in rs]),
                    best_restart=np.array([r["best_restart"] for r in rs]),
                    best_x=np.concatenate([r["best_x"] for r in rs]))
    if kind == "lagr":
        L = pdbo.MaxSATLagrangian.apply(state["x"], state["y"], ctx)
        dx, dy = torch.autograd.grad(L, (state["x"], state["y"]), state["w"])
        return dict(L=L.detach(), dx=dx, dy=dy)
    if kind == "dual":
        return pdbo.qubo_dual_bound(ctx, case["iters"])
    return pdbo.qubo_gda_eval_noalloc(ctx, state["xr"], state["F"])


# ---------------------------------------------------------------- work


def _nnz(case):
    return int(case["n"] * case["deg"])


def work(case):
    kind = case["kind"]
    n, B = case.get("n", 0), case["B"]
    eb = {"fp32": 4, "bf16": 2, "i8": 1, "fp8": 1}[case.get("prec", "fp32")]

    def iterated(matrix, state, flops, T):
        # what fits in the chip's LDS (256 x 160 KB) is read once, the rest every iteration
        per = (matrix if matrix > 40e6 else 0) + (2 * state if state > 40e6 else 0)
        return dict(bytes=float(matrix + 2 * state + T * per), flops=float(T * flops))

    if kind == "solve":
        fam, T = case["family"], case["T"]
        if fam == "dense":
            return iterated(eb * n * n, 8 * n * B, 2.0 * n * n * B, T)
        if fam in ("csr", "mis"):
            return iterated(4 * _nnz(case), 8 * n * B, 2.0 * _nnz(case) * B, T)
        if fam == "kcut":
            return iterated(4 * _nnz(case), 4 * (case["k"] + 1) * n * B, 2.0 * case["k"] * _nnz(case) * B, T)
        m, k = int(n * case["ratio"]), case["k"]
        return iterated(4 * m * k, 8 * n * B, 2.0 * k * k * m * B, T)
    if kind == "batch":
        lo, hi = case["lo"], case["hi"]
        mean, sq = (lo + hi) / 2.0, (lo * lo + lo * hi + hi * hi) / 3.0
        return iterated(case["count"] * eb * sq, case["count"] * 8 * mean * B, 2.0 * case["count"] * sq * B, case["T"])
    if kind == "lagr":
        m, k = int(n * case["ratio"]), case["k"]
        return dict(bytes=float(16 * n * B + 8 * B + 4 * m * k), flops=float(2 * m * k * k * B))
    if kind == "dual":
        return iterated(eb * n * n, 8 * n, 2.0 * n * n, case["iters"])
    fam = case["family"]
    size = {"dense": lambda: n * n, "csr": lambda: _nnz(case), "kcut": lambda: _nnz(case),
            "sat": lambda: int(n * case["ratio"]) * case["k"]}[fam]()
    return dict(bytes=float(n * B + size + 8 * B), flops=float(2.0 * size * B))


# ---------------------------------------------------------------- float64


def _philox(seed, B, n):
    """Philox4x32-10 starting points (Salmon et al., SC 2011): coordinate i of
    restart b is word i mod 4 for the counter (i div 4, b, 0, 0)."""
    q = (n + 3) // 4
    mask = np.uint64(0xFFFFFFFF)
    c = [np.broadcast_to(np.arange(q, dtype=np.uint64)[None], (B, q)),
         np.broadcast_to(np.arange(B, dtype=np.uint64)[:, None], (B, q)),
         np.zeros((B, q), np.uint64), np.zeros((B, q), np.uint64)]
    k = [seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF]
    for r in range(10):
        if r:
            k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k[0]), p1 & mask,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k[1]), p0 & mask]
    w = np.stack(c, axis=2).reshape(B, 4 * q)[:, :n]
    return (w >> np.uint64(8)).astype(np.float64) * 2.0 ** -24


def _g(x, kind):
    if kind == "quad":
        return x * x - x, 2 * x - 1
    e = 2.0 ** -20
    v = torch.special.xlogy(x, x) + torch.special.xlogy(1 - x, 1 - x)
    xc = x.clamp(e, 1 - e)
    return v, torch.log(xc) - torch.log1p(-xc)


def _descend(product, lin, x, y, p, T):
    """T iterations of Alg. 1 in float64; x, y are (B, n)."""
    for _ in range(T):
        gv, gd = _g(x, p["g"])
        dL = product(x) + lin + y * gd
        pert = ((x - 0.5).abs() <= p["delta"]) & (dL.abs() <= 2 * p["delta"]) & (y <= 0)
        moved = torch.where(x <= 0.5, 0.5 - p["delta"], 0.5 + p["delta"])
        x, y = torch.where(pert, moved, (x - p["alpha"] * dL).clamp(0, 1)), y + p["beta"] * gv
    return x, y


def _canonical(inst, scale):
    """x -> A x / s and c' / s of the canonical form, in float64 on the GPU."""
    n = inst.n
    if inst.Q is not None:
        Q = torch.from_numpy(inst.Q).cuda().double()
    else:
        Q = torch.zeros((n, n), dtype=torch.float64, device="cuda")
        rows = torch.from_numpy(np.repeat(np.arange(n), np.diff(inst.row_ptr))).cuda()
        Q[rows, torch.from_numpy(inst.col_idx).cuda().long()] = torch.from_numpy(inst.vals).cuda().double()
    d = torch.diagonal(Q).clone()
    A = (Q + Q.T)
    A.fill_diagonal_(0)
    A /= scale
    c = d if inst.c is None else d + torch.from_numpy(inst.c).cuda().double()
    return A, c / scale


def _sat_parts(inst, scale):
    """x (B, n) -> f(x)/s (B,) and its gradient (B, n)."""
    lits = torch.from_numpy(inst.lits).cuda().long()
    var, neg = lits.abs() - 1, lits < 0
    cw = torch.from_numpy(inst.w).cuda().double() / scale

    def parts(x):
        f, grad = torch.zeros(len(x), dtype=x.dtype, device=x.device), torch.zeros_like(x)
        for b in range(0, len(x), 8):
            xv = x[b:b + 8][:, var]
            p = torch.where(neg, xv, 1 - xv)
            f[b:b + 8] = (cw * p.prod(2)).sum(1)
            for l in range(var.shape[1]):
                others = torch.cat([p[:, :, :l], p[:, :, l + 1:]], 2).prod(2)
                grad[b:b + 8].index_add_(1, var[:, l], cw * torch.where(neg[:, l], others, -others))
        return f, grad

    return parts


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve" and case["state"] and case["family"] == "sat":
        inst, scale = _sat(case, seed)
        parts, p = _sat_parts(inst, scale), _params(case, "sat", scale, seed)
        x = torch.from_numpy(_philox(seed, case["B"], case["n"])).cuda()
        x, y = _descend(lambda v: parts(v)[1], 0.0, x, torch.full_like(x, p["y0"]), p, case["T"])
        return dict(best_obj=None, best_restart=None, best_iter=None, best_x=None, F=None, x=x, y=y)
    if kind == "solve" and case["state"] and case["family"] in ("dense", "csr"):
        inst, scale = _MAKE[case["family"]](case, seed)
        A, lin = _canonical(inst, scale)
        p = _params(case, case["family"], scale, seed)
        x = torch.from_numpy(_philox(seed, case["B"], case["n"])).cuda()
        x, y = _descend(lambda v: v @ A, lin, x, torch.full_like(x, p["y0"]), p, case["T"])
        out = dict(best_obj=None, best_restart=None, best_iter=None, best_x=None, F=None, x=x, y=y)
        return out
    if kind == "lagr":
        inst, scale = _sat(case, seed)
        x, y, w = (t.double() for t in _lagr_inputs(case, seed))
        gv, gd = _g(x, case["g"])
        f, grad = _sat_parts(inst, scale)(x)
        L, dx = f + (y * gv).sum(1), grad + y * gd
        return dict(L=L, dx=w[:, None] * dx, dy=w[:, None] * gv)
    if kind == "dual":
        inst, scale = _dense_qubo(case, seed)
        A, lin = _canonical(inst, scale)
        p = _params(case, "dense", scale, seed)
        x = torch.full((1, case["n"]), 0.5, dtype=torch.float64, device="cuda")
        x, _ = _descend(lambda v: v @ A, lin, x, torch.full_like(x, p["y0"]), dict(p, beta=0.0), case["iters"])
        Ax = x @ A
        d = Ax + lin + p["y0"] * (2 * x - 1)
        value = scale * float((x * (0.5 * Ax + lin) + p["y0"] * (x * x - x)).sum())
        gap = scale * float(-torch.minimum(-d * x, d * (1 - x)).sum())
        return dict(lower_bound=value - gap, value=value, gap=None, rounding=None, x=x[0])
    return None
