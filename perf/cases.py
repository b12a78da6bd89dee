"""What the library's performance is measured on: scoring passes, training and
serving at the sizes of this repository's tests and benchmark and around them.

A case names an operation and its sizes: ``K`` profiled kernels with ``lo`` to
``hi`` of ``D`` optimisations each (all 2^B versions of every kernel), ``E``
counter events, ``dtype`` "f32" or "f64".  Inputs follow the synthetic world
of the tests (lognormal counters, speedups linear in the log-rates plus
pairwise interactions and noise), drawn on the GPU from the seed.  A batch's
structure (how many optimisations each kernel has, and which) depends on the
case alone.
"""
import math

import numpy as np
import torch

from paper_1910_07776_amd import plain as G
from paper_1910_07776_amd.surrogate import MLP

DEV = "cuda"
DT = {"f32": torch.float32, "f64": torch.float64}
HIDDEN = 512
TOL, BAND, CAP = 0.1, 0.1, 16          # a serving query's defaults
LR, STEPS0 = 1e-3, 1000


def listed():
    return [
        # two small programs compared against each other in double precision: the smallest call, all latency
        dict(name="suggest_pair_f64", op="suggest", K=2, lo=6, hi=6, D=6, E=40, dtype="f64"),
        # an ordinary batch: 512 kernels with all 64 versions of six optimisations
        dict(name="suggest_512", op="suggest", K=512, lo=6, hi=6, D=6, E=128, dtype="f32"),
        # the benchmark's headline: a ragged batch of 16,384 kernels, 4.8 million versions
        dict(name="suggest_ragged_16384", op="suggest", K=16384, lo=4, hi=10, D=10, E=128, dtype="f32"),
        # every single-optimisation prediction of a ragged batch with an odd number of events
        dict(name="grid_ragged_1000", op="grid", K=1000, lo=4, hi=10, D=10, E=100, dtype="f32"),
        # the estimate that does not depend on the order of the optimisations
        dict(name="allpaths_512", op="allpaths", K=512, lo=6, hi=6, D=6, E=128, dtype="f32"),
        # training of the linear models on the ordinary batch, and its checkpoint
        dict(name="fit_512", op="fit", K=512, lo=6, hi=6, D=6, E=128, dtype="f32"),
        # the same on the benchmark's training set
        dict(name="fit_ragged_16384", op="fit", K=16384, lo=4, hi=10, D=10, E=128, dtype="f32"),
        # nearest-neighbour models from 512 training kernels scoring 512 others
        dict(name="ibk_512", op="ibk", K=512, lo=6, hi=6, D=6, E=128, dtype="f32", train=512, k=10),
        # model trees scoring an ordinary batch
        dict(name="m5p_512", op="m5p", K=512, lo=6, hi=6, D=6, E=128, dtype="f32", train=64),
        # training of the surrogate network: mini-batches of 4096 kernels out of 65,536
        dict(name="train_4096", op="train", rows=65536, batch=4096, steps=8, E=128, B=6),
        # the surrogate's answer for a large batch (one pass of the network and its ranking)
        dict(name="surrogate_65536", op="surrogate", K=65536, lo=6, hi=6, D=6, E=128, dtype="f32"),
        # the largest serving query: 4096 kernels with 1024 versions each, judged by the linear models
        dict(name="serve_4096x1024", op="serve", K=4096, lo=10, hi=10, D=10, E=128, dtype="f32"),
    ]


def _log_int(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    op = rng.choice(["suggest"] * 4 + ["grid", "allpaths", "fit", "fit", "ibk", "ibk", "m5p", "train", "surrogate",
                                       "serve", "serve"])
    if op == "train":
        batch = _log_int(rng, 100, 4096)
        return dict(op=op, rows=batch * rng.randint(2, 16), batch=batch, steps=rng.randint(2, 8), E=128,
                    B=rng.choice([6, 6, 7]))
    if op in ("surrogate", "serve"):
        B = 6 if op == "surrogate" else rng.randint(6, 10)
        most = 65536 if op == "surrogate" else 4096
        return dict(op=op, K=_log_int(rng, 1, most), lo=B, hi=B, D=B if op == "surrogate" else 10,
                    E=rng.choice([40, 128, 128]), dtype="f32")
    E = rng.choice([40, 128, 128, rng.randint(17, 256)])
    if rng.random() < 0.5:
        B = rng.randint(4, 8)
        D, lo, hi = B, B, B
    else:
        D, lo, hi = 10, 4, rng.randint(6, 10)
    mean_rows = sum(1 << b for b in range(lo, hi + 1)) / (hi - lo + 1)
    most = {"suggest": 4.0e6, "grid": 3.0e5, "allpaths": 3.0e5, "fit": 2.0e6, "ibk": 3.2e4, "m5p": 6.0e4}[op]
    if E > 128:
        most /= 2
    K = _log_int(rng, 64 if op == "fit" else 1, max(65 if op == "fit" else 1, min(16384, most / mean_rows)))
    c = dict(op=op, K=K, lo=lo, hi=hi, D=D, E=E, dtype="f64" if rng.random() < 0.2 and K * mean_rows < 3e5 else "f32")
    if op == "ibk":
        c.update(train=_log_int(rng, 24, 512 * 64 / mean_rows), k=rng.choice([3, 5, 10, 10]), E=min(E, 128))
    if op == "m5p":
        c.update(train=_log_int(rng, 24, 64))
    return c


# ---- inputs -------------------------------------------------------------------
def _structure(K, lo, hi, D, salt=0):
    """Optimisation counts, which of the D ids each kernel has, and the flat id list."""
    r = np.random.default_rng([K, lo, hi, D, salt])
    nopts = r.integers(lo, hi + 1, size=K).astype(np.int32)
    has = np.argsort(np.argsort(r.random((K, D)), axis=1), axis=1) < nopts[:, None]
    return nopts, has, np.nonzero(has)[1].astype(np.int32)


def _bits(nopts, has):
    """Per row (version): its kernel and which global ids it has applied."""
    n = torch.from_numpy(np.left_shift(1, nopts.astype(np.int64))).to(DEV)
    kern = torch.repeat_interleave(torch.arange(len(nopts), device=DEV), n)
    off = torch.cumsum(n, 0) - n
    S = torch.arange(int(n.sum()), device=DEV) - off[kern]
    h = torch.from_numpy(has).to(DEV)
    pos = torch.cumsum(h.to(torch.int64), 1) - 1
    bits = torch.stack([h[:, o][kern] & (((S >> pos[:, o][kern].clamp(min=0)) & 1) == 1) for o in range(has.shape[1])],
                       1)
    return kern, S, bits


class _World:
    """Column means, effects of the optimisations on speedup and counters."""

    def __init__(self, seed, E, D):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(1000003 * int(seed) + 17)
        self.E, self.D = E, D
        r = np.random.default_rng([int(seed), E, D])
        f = lambda a: torch.as_tensor(a, dtype=torch.float64, device=DEV)  # noqa: E731
        self.mu = f(r.uniform(2.0, 12.0, E + 1))
        self.bias = f(r.uniform(-0.05, 0.20, D))
        self.w = f(r.normal(0.0, 0.15 / math.sqrt(E), (D, E)))
        pair = np.triu(r.normal(0.0, 0.03, (D, D)), 1)
        self.pair = f(pair + pair.T)
        self.delta = f(r.normal(0.0, 0.1, (D, E)))

    def batch(self, nopts, has, dtype):
        """Counters [N, E] and cycles [N] of a batch."""
        kern, S, bits = _bits(nopts, has)
        K, E, g = len(nopts), self.E, self.g
        lc0 = self.mu + 0.5 * torch.randn((K, E + 1), generator=g, device=DEV, dtype=torch.float64)
        u = (lc0[:, :E] - self.mu[:E] - (lc0[:, E:] - self.mu[E:])) * math.sqrt(2.0)
        lin = u @ self.w.T + self.bias
        fb = bits.to(torch.float64)
        T = (fb * lin[kern]).sum(1) + 0.5 * ((fb @ self.pair) * fb).sum(1)
        T += 0.05 * torch.randn(T.shape, generator=g, device=DEV, dtype=torch.float64) * (S > 0)
        counters = torch.randn((len(kern), E), generator=g, device=DEV, dtype=dtype)
        counters.mul_(0.02).add_(lc0[:, :E].to(dtype)[kern]).add_(bits.to(dtype) @ self.delta.to(dtype)).exp_()
        return counters, torch.exp(lc0[kern, E] - T).to(dtype)


def _plan(ctx, case, s):
    return G.Plan(ctx, s[0], s[2], case["E"], case["D"], dtype=DT[case["dtype"]])


def _train_structure(case):
    """Training kernels of the models a scoring case uses."""
    D, lo, hi = case["D"], case["lo"], case["hi"]
    K = case.get("train") or (128 if case["op"] == "serve" else 256)
    return _structure(K, min(hi, max(lo, 6)), hi, D, salt=1)


def _inputs(case, seed):
    """The world, the training set and the batch, in the order that fixes the draw."""
    w = _World(seed, case["E"], case["D"])
    tr = te = None
    if case["op"] != "fit":
        st = _train_structure(case)
        tr = (st, *w.batch(st[0], st[1], DT[case["dtype"]]))
    s = _structure(case["K"], case["lo"], case["hi"], case["D"])
    te = (s, *w.batch(s[0], s[1], DT[case["dtype"]]))
    return w, tr, te


def _net(w, E, A, b):
    """Parameters of an in-512-512-out network that computes z A^T + b through
    its two GELU layers (gelu(t) - gelu(-t) = t), with dense weights: what a
    trained surrogate of a linear table computes."""
    h = HIDDEN // 2
    gauss = lambda m, n: torch.randn((m, n), generator=w.g, device=DEV, dtype=torch.float64)  # noqa: E731
    Q = torch.linalg.qr(gauss(h, E))[0]
    R = torch.linalg.qr(gauss(h, h))[0]
    W1 = torch.cat([Q, -Q])
    W2 = torch.cat([torch.cat([R, -R], 1), torch.cat([-R, R], 1)])
    M = A @ Q.T @ R.T
    W3 = torch.cat([M, -M], 1)
    zero = torch.zeros(HIDDEN, device=DEV, dtype=torch.float64)
    return torch.cat([t.reshape(-1) for t in (W1, zero, W2, zero, W3, b)]).float()


def _surrogate_params(w, tr, case):
    """Parameters fitted to the linear models' tables of 512 other kernels, off
    by a few hundredths as a trained network's are."""
    B, E = case["lo"], case["E"]
    s = _structure(512, B, B, B)
    has = np.zeros((512, case["D"]), bool)
    has[:, :B] = True
    c, cyc = w.batch(s[0], has, torch.float32)
    mu, sg, W = _fit(*tr, E, case["D"])
    z = _z(c, cyc, mu, sg)
    Y = _chain(s, torch.addmm(W[:, E], z, W[:, :E].T)).view(512, 1 << B)
    X = z[::1 << B]
    m = Y.mean(0)
    A = torch.linalg.solve(X.T @ X + torch.eye(E, device=DEV, dtype=torch.float64), X.T @ (Y - m)).T
    A = A + 0.03 / math.sqrt(E) * torch.randn(A.shape, generator=w.g, device=DEV, dtype=torch.float64)
    return _net(w, E, A, m - X.mean(0) @ A.T)


def prepare(case, seed):
    op = case["op"]
    st = {"case": dict(case), "ctx": G.Context(0)}
    ctx = st["ctx"]
    if op == "train":
        g = torch.Generator(device=DEV)
        g.manual_seed(7919 * int(seed) + 3)
        E, out = case["E"], 1 << case["B"]
        p, st["X"], st["Y"], st["perm"], m, v = _train_inputs(case, g)
        mlp = st["mlp"] = MLP(ctx, E, HIDDEN, out, max_batch=case["batch"], params=p.cpu().numpy())
        mlp.m.copy_(m)
        mlp.v.copy_(v)
        mlp.step = STEPS0
        return st
    w, tr, te = _inputs(case, seed)
    if tr is not None:
        train = _plan(ctx, case, tr[0])
        if op == "ibk":
            G.ibk_fit(ctx, train, tr[1], tr[2], k=case["k"])
        elif op == "m5p":
            G.m5p_fit(ctx, train, tr[1], tr[2])
        else:
            G.fit(ctx, train, tr[1], tr[2])
    s = te[0]
    if op in ("surrogate", "serve"):   # the kernels of a query have the first B optimisations
        K, B = case["K"], case["lo"]
        mlp = MLP(ctx, case["E"], HIDDEN, 1 << B, max_batch=max(64, K),
                  params=_surrogate_params(w, tr, case).cpu().numpy())
        st["mlp"] = mlp.freeze()
        if op == "serve":
            has = np.zeros((K, case["D"]), bool)
            has[:, :B] = True
            s = (s[0], has, np.tile(np.arange(B, dtype=np.int32), K))
            te = (s, *w.batch(s[0], has, torch.float32))
    st["plan"], st["counters"], st["cycles"] = _plan(ctx, case, s), te[1], te[2]
    G.sync(ctx)
    return st


def _train_inputs(case, g):
    """Parameters, features, target tables, the epoch's order and Adam's moments midway."""
    E, out, n = case["E"], 1 << case["B"], case["rows"]
    p = torch.cat([(2.0 * torch.rand(fo * (fi + 1), generator=g, device=DEV) - 1.0) / math.sqrt(fi)
                   for fi, fo in ((E, HIDDEN), (HIDDEN, HIDDEN), (HIDDEN, out))])
    P = p.numel()
    X = torch.randn((n, E), generator=g, device=DEV)
    Y = 0.3 * (X @ (torch.randn((E, out), generator=g, device=DEV) / math.sqrt(E))) + 0.2
    perm = torch.randperm(n, generator=g, device=DEV)[:case["batch"] * case["steps"]].to(torch.int32)
    m = 1e-4 * torch.randn(P, generator=g, device=DEV)
    v = 1e-6 * (0.1 + torch.rand(P, generator=g, device=DEV))
    return p, X, Y, perm, m, v


def run(st):
    case, ctx = st["case"], st["ctx"]
    op = case["op"]
    if op == "train":
        mlp = st["mlp"]
        losses = mlp.train_epoch(st["X"], st["Y"], st["perm"], case["batch"], LR)
        return {"losses": losses, "params": mlp.params, "grads": mlp.grads, "m": mlp.m, "v": mlp.v}
    plan, c, cyc = st["plan"], st["counters"], st["cycles"]
    if op == "fit":
        G.fit(ctx, plan, c, cyc)
        return ctx.model_get()
    if op == "grid":
        table, grid = G.predict(ctx, plan, c, cyc, grid=True)
        return {"table": table, "grid": grid}
    if op == "allpaths":
        table, idx, score, count = G.predict_allpaths(ctx, plan, c, cyc)
    elif op == "surrogate":
        idx, score, count, table = G.surrogate_suggest(ctx, plan, st["mlp"], c, cyc, table=True)
    elif op == "serve":
        K = plan.K
        out = {"idx": torch.empty((K, 3), dtype=torch.int32, device=DEV),
               "score": torch.empty((K, 3), device=DEV), "count": torch.empty(K, dtype=torch.int32, device=DEV)}
        flag = torch.empty(K, dtype=torch.int32, device=DEV)
        G.serve_query(ctx, plan, st["mlp"], c, cyc, out, flag, tol=TOL, band=BAND, cap=CAP)
        return dict(out, flag=flag)
    else:
        f = {"suggest": G.suggest, "ibk": G.ibk_suggest, "m5p": G.m5p_suggest}[op]
        idx, score, count, table = f(ctx, plan, c, cyc)
    return {"idx": idx, "score": score, "count": count, "table": table}


# ---- what a pass cannot do without --------------------------------------------
def work(case):
    op = case["op"]
    if op == "train":
        E, out, n = case["E"], 1 << case["B"], case["batch"] * case["steps"]
        P = E * HIDDEN + HIDDEN * HIDDEN + HIDDEN * out
        # inputs and targets once; parameters, gradients and both moments read and written by every step
        return {"bytes": 4.0 * n * (E + out) + 28.0 * P * case["steps"], "flops": 6.0 * n * P - 2.0 * n * E * HIDDEN}
    E, K, ts = case["E"], case["K"], 8 if case["dtype"] == "f64" else 4
    nopts, has, ids = _structure(K, case["lo"], case["hi"], case["D"])
    N = int(np.left_shift(1, nopts.astype(np.int64)).sum())
    rows = float(N) * (E + 1) * ts
    lists = K * 3 * (4 + ts) + 4.0 * K
    if op == "fit":   # every row's outer product once
        return {"bytes": rows + 8.0 * case["D"] * (E + 1), "flops": float(N) * E * (E + 1)}
    if op == "grid":
        return {"bytes": rows + N * ts * (1.0 + int(nopts.max())), "flops": N * E * (3.0 + float(nopts.mean()))}
    if op == "allpaths":
        return {"bytes": rows + N * ts + lists, "flops": N * E * (3.0 + float(nopts.mean()))}
    if op == "surrogate":
        P = E * HIDDEN + HIDDEN * HIDDEN + HIDDEN * 64
        return {"bytes": K * (E + 1 + 64) * 4.0 + lists + 2.0 * P, "flops": 2.0 * K * P}
    if op == "serve":   # baseline rows, the network, and the listed subsets' chains (about half of B rows each)
        B = case["lo"]
        P = E * HIDDEN + HIDDEN * HIDDEN + HIDDEN * (1 << B)
        return {"bytes": K * (1 + 3 * B / 2) * (E + 1) * 4.0 + lists + 4.0 * K + 2.0 * P, "flops": 2.0 * K * P}
    if op == "ibk":   # the distance of every query to every stored sample of its optimisation
        tn, th, _ = _train_structure(case)
        samples = (th * np.left_shift(1, tn.astype(np.int64) - 1)[:, None]).sum(0)
        local = np.cumsum(has, 1) - 1
        queries = np.where(has, np.left_shift(1, local.clip(0)), 0).sum(0)
        trows = float(np.left_shift(1, tn.astype(np.int64)).sum())
        return {"bytes": rows + trows * E * ts + N * ts + lists, "flops": 2.0 * E * float((samples * queries).sum())}
    return {"bytes": rows + N * ts + lists, "flops": N * E * 5.0}


# ---- the same in 64 bits -------------------------------------------------------
def _z(c, cyc, mu, sg):
    return (torch.log(c.double()) - torch.log(cyc.double())[:, None] - mu) / sg


def _stats(c, cyc):
    x = torch.log(c.double()) - torch.log(cyc.double())[:, None]
    mu = x.mean(0)
    sg = ((x - mu) ** 2).mean(0).sqrt()
    return mu, torch.where(sg < 1e-12, torch.ones_like(sg), sg)


def _pairs(s):
    """Per global id: before rows and after rows of every pair (kernel order, versions ascending)."""
    nopts, has, _ = s
    kern, S, bits = _bits(nopts, has)
    h = torch.from_numpy(has).to(DEV)
    pos = torch.cumsum(h.to(torch.int64), 1) - 1
    for o in range(has.shape[1]):
        before = torch.nonzero(h[:, o][kern] & ~bits[:, o]).flatten()
        yield o, before, before + (1 << pos[kern[before], o])


def _fit(s, c, cyc, E, D, lam=1e-2):
    mu, sg = _stats(c, cyc)
    z, lc = _z(c, cyc, mu, sg), torch.log(cyc.double())
    W = torch.full((D, E + 1), math.nan, device=DEV, dtype=torch.float64)
    pen = torch.full((E + 1,), lam, device=DEV, dtype=torch.float64)
    pen[E] = 0.0
    for o, b, a in _pairs(s):
        if not len(b):
            continue
        A = torch.diag(pen)
        r = torch.zeros(E + 1, device=DEV, dtype=torch.float64)
        for i in range(0, len(b), 1 << 18):
            q = b[i:i + (1 << 18)]
            x = torch.cat([z[q], torch.ones((len(q), 1), device=DEV, dtype=torch.float64)], 1)
            A += x.T @ x
            r += x.T @ (lc[q] - lc[a[i:i + (1 << 18)]])
        W[o] = torch.linalg.solve(A, r)
    return mu, sg, W


def _by_B(s):
    """(B, first rows [n], ids [n, B]) of the kernels of each B."""
    nopts, _, ids = s
    off = np.concatenate([[0], np.cumsum(np.left_shift(1, nopts.astype(np.int64)))])[:-1]
    io = np.concatenate([[0], np.cumsum(nopts)])[:-1]
    for B in sorted(set(nopts.tolist())):
        k = np.nonzero(nopts == B)[0]
        yield (B, torch.from_numpy(k).to(DEV), torch.from_numpy(off[k]).to(DEV),
               torch.from_numpy(ids[io[k][:, None] + np.arange(B)].astype(np.int64)).to(DEV))


def _scores(s, table, tau=G.TAU, n=3):
    out = torch.full((len(s[0]), n), math.nan, device=DEV, dtype=torch.float64)
    for B, k, off, _ in _by_B(s):
        t = table[off[:, None] + torch.arange(1 << B, device=DEV)].clone()
        t[:, 0] = -math.inf
        t[t <= tau] = -math.inf
        v = torch.topk(t, min(n, 1 << B), dim=1).values
        out[k, :v.shape[1]] = torch.where(torch.isinf(v), math.nan, v)
    return out


def _chain(s, P):
    """Composed table from P [N, D] (prediction of adding id o to the row's version)."""
    table = torch.zeros(P.shape[0], device=DEV, dtype=torch.float64)
    for B, _, off, ids in _by_B(s):
        for b in range(B):
            lo = torch.arange(1 << b, device=DEV)
            r = off[:, None] + lo
            table[r + (1 << b)] = table[r] + P[r, ids[:, b:b + 1].expand(-1, 1 << b)]
    return table


def _allpaths(s, P):
    table = torch.zeros(P.shape[0], device=DEV, dtype=torch.float64)
    for B, _, off, ids in _by_B(s):
        S = torch.arange(1 << B, device=DEV)
        ones = sum((S >> b) & 1 for b in range(B)) if B else S
        for level in range(1, B + 1):
            at = S[ones == level]
            acc = torch.zeros((len(off), len(at)), device=DEV, dtype=torch.float64)
            for b in range(B):
                on = ((at >> b) & 1) == 1
                r = off[:, None] + (at[on] - (1 << b))
                acc[:, on] += table[r] + P[r, ids[:, b:b + 1].expand(-1, int(on.sum()))]
            table[off[:, None] + at] = acc / level
    return table


def exact(case, seed):
    op, E = case["op"], case["E"]
    if op in ("m5p", "serve"):
        return None   # the trees' induction, and lists that hang on the network's rounding
    if op == "train":
        return _exact_train(case, seed)
    w, tr, te = _inputs(case, seed)
    s, c, cyc = te
    if op == "fit":
        mu, sg, W = _fit(s, c, cyc, E, case["D"])
        return {"mu": mu, "sigma": sg, "W": W, "counts": None}
    if op == "ibk":
        P = _exact_ibk(case, tr, te)
        table = _chain(s, P)
        return {"idx": None, "score": _scores(s, table), "count": None, "table": table}
    mu, sg, W = _fit(*tr, E, case["D"])
    if op == "surrogate":
        p = _surrogate_params(w, tr, case).double()
        x = _z(c[::64], cyc[::64], mu, sg)
        table = _mlp(p, x, E, 64)
        return {"idx": None, "score": None, "count": None, "table": table}
    P = torch.addmm(W[:, E], _z(c, cyc, mu, sg), W[:, :E].T)
    if op == "grid":
        grid = torch.full((len(c), int(s[0].max())), math.nan, device=DEV, dtype=torch.float64)
        for B, _, off, ids in _by_B(s):
            S = torch.arange(1 << B, device=DEV)
            for b in range(B):
                r = off[:, None] + S[((S >> b) & 1) == 0]
                grid[r, b] = P[r, ids[:, b:b + 1].expand(-1, r.shape[1])]
        return {"table": _chain(s, P), "grid": grid}
    table = _allpaths(s, P) if op == "allpaths" else _chain(s, P)
    return {"idx": None, "score": _scores(s, table), "count": None, "table": table}


def _exact_ibk(case, tr, te):
    """Mean label of the k nearest stored samples, for every row and id that a chain asks for."""
    mu, sg = _stats(tr[1], tr[2])
    zt, zq, lc = _z(tr[1], tr[2], mu, sg), _z(te[1], te[2], mu, sg), torch.log(tr[2].double())
    P = torch.zeros((len(zq), case["D"]), device=DEV, dtype=torch.float64)
    need = torch.zeros((len(zq), case["D"]), device=DEV, dtype=torch.bool)
    for B, _, off, ids in _by_B(te[0]):
        for b in range(B):
            r = off[:, None] + torch.arange(1 << b, device=DEV)
            need[r, ids[:, b:b + 1].expand(-1, 1 << b)] = True
    for o, before, after in _pairs(tr[0]):
        q = torch.nonzero(need[:, o]).flatten()
        t, y = zt[before], lc[before] - lc[after]
        for i in range(0, len(q), 2048):
            x = zq[q[i:i + 2048]]
            d = (x * x).sum(1)[:, None] + (t * t).sum(1) - 2.0 * (x @ t.T)
            near = torch.topk(d, min(case["k"], len(t)), dim=1, largest=False).indices
            P[q[i:i + 2048], o] = y[near].mean(1)
    return P


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x * math.sqrt(0.5)))


def _mlp(p, x, E, out):
    k = 0
    for i, (fi, fo) in enumerate(((E, HIDDEN), (HIDDEN, HIDDEN), (HIDDEN, out))):
        Wl, bl = p[k:k + fi * fo].view(fo, fi), p[k + fi * fo:k + fi * fo + fo]
        k += fi * fo + fo
        x = torch.addmm(bl, x, Wl.T)
        if i < 2:
            x = _gelu(x)
    return x


def _exact_train(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(7919 * int(seed) + 3)
    E, out = case["E"], 1 << case["B"]
    p, X, Y, perm, m, v = _train_inputs(case, g)
    p, m, v = p.double(), m.double(), v.double()
    losses, n = [], case["batch"]
    for i in range(case["steps"]):
        q = perm[i * n:(i + 1) * n].long()
        pp = p.clone().requires_grad_(True)
        loss = ((_mlp(pp, X[q].double(), E, out) - Y[q].double()) ** 2).mean()
        loss.backward()
        losses.append(loss.detach())
        t = STEPS0 + i + 1
        m = 0.9 * m + 0.1 * pp.grad
        v = 0.999 * v + 0.001 * pp.grad ** 2
        p = p - LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return {"losses": torch.stack(losses), "params": p, "grads": pp.grad, "m": m, "v": v}
