"""The serving query against the same steps taken one by one through the
library's public calls (inference, ranking, band, judge, masked plain pass)
and Tier 3's contract in numpy: identical answers and flags, at table widths
on both sides of the output layer's own ranking, full, short and empty lists,
bands over their cap, and counters that are not aligned for wide loads."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TAU = 0.02


@pytest.mark.parametrize("B,E,K,n,cap,tol,band,shift", [
    (3, 40, 5, 3, 1, 0.3, 0.1, 0), (6, 128, 700, 3, 16, 0.3, 0.05, 0), (7, 128, 130, 8, 64, 9.0, 0.02, 1),
    (8, 40, 600, 3, 4, 9.0, 0.03, 0), (8, 200, 64, 1, 16, 0.2, 0.05, 0), (9, 128, 257, 8, 2, 9.0, 0.03, 1),
    (10, 128, 300, 3, 16, 0.3, 0.05, 0), (12, 64, 3, 5, 64, 9.0, 0.04, 0)])
def test_query_equals_its_steps(B, E, K, n, cap, tol, band, shift):
    from paper_1910_07776_amd import plain as G, surrogate as S
    from synthgen import make_batch
    ctx = G.Context(0, n_suggest=n, tau=TAU)
    V, D = 1 << B, 12
    tr = make_batch(91, range(100, 228), E, D, brange=(0, 8))
    G.fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D), torch.from_numpy(tr.counters).cuda(),
          torch.from_numpy(tr.cycles).cuda())
    te = make_batch(91, range(1000, 1000 + K), E, D, brange=(B, B))
    assert (te.nopts == B).all()
    p = G.Plan(ctx, te.nopts, te.opt_ids, E, D)
    buf = torch.empty(te.N * E + shift, device="cuda")
    c = buf[shift:].view(te.N, E)      # shift 1: rows not aligned to 16 bytes
    c.copy_(torch.from_numpy(te.counters))
    cy = torch.from_numpy(te.cycles).float().cuda()
    mlp = S.MLP(ctx, E, 512, V, max_batch=K, seed=92)
    u = mlp.unflatten(mlp.params)
    rng = np.random.default_rng(93)
    # about two columns near and above the threshold, a few within the band
    b3 = np.where(rng.random(V) < 2.0 / V, 0.03, np.where(rng.random(V) < 6.0 / V, 0.0, -0.2))
    u["b3"].copy_(torch.from_numpy(b3.astype(np.float32)))
    u["W3"].mul_(0.3)
    mlp.freeze()
    out = {"idx": torch.full((K, n), -9, dtype=torch.int32, device="cuda"),
           "score": torch.full((K, n), -9.0, device="cuda"),
           "count": torch.full((K,), -9, dtype=torch.int32, device="cuda")}
    flag = torch.full((K,), -9, dtype=torch.int32, device="cuda")
    G.serve_query(ctx, p, mlp, c, cy, out, flag, tol=tol, band=band, cap=cap)
    idx, sc, cnt = out["idx"], out["score"], out["count"]

    zz = G.load_features(ctx, p, c, cy, baseline=True)
    y = mlp.infer(zz)
    seg = torch.arange(0, K + 1, dtype=torch.int64, device="cuda") * V
    ri, rs, rc = G.rank_suggest(ctx, y.view(-1), seg, n=n, tau=TAU, skip_head=1)
    bi, br, fl = G.band_select(ctx, y.view(-1), seg, ri, rc, tau=TAU, band=band, cap=cap, skip_head=1)
    pl = G.judge(ctx, p, c, cy, ri, ref=rs, tol=tol, flag=fl, accumulate=True)
    pb = G.judge(ctx, p, c, cy, bi, ref=br, tol=tol, flag=fl, accumulate=True)
    G.sync(ctx)
    ri, rc, bi, fl, pl, pb = (x.cpu().numpy() for x in (ri, rc, bi, fl, pl, pb))
    tau = np.float32(TAU)
    want_i, want_s = ri.copy(), pl.copy()
    for k in range(K):
        if not fl[k] and (not (pl[k, :rc[k]] > tau).all() or (pb[k][bi[k] >= 0] > tau).any()):
            fl[k] = 1
        if not fl[k]:
            o = np.lexsort((ri[k, :rc[k]], -pl[k, :rc[k]]))
            want_i[k, :rc[k]], want_s[k, :rc[k]] = ri[k][o], pl[k][o]
    full_i, full_s, full_c, _ = G.suggest(ctx, p, c, cy)
    G.sync(ctx)
    f = fl.astype(bool)
    want_i[f], want_s[f], rc[f] = full_i.cpu().numpy()[f], full_s.cpu().numpy()[f], full_c.cpu().numpy()[f]
    print(f"B {B}: flagged {f.mean():.2f}, listed {rc.mean():.2f}, band {(bi >= 0).sum(1).mean():.2f}")
    assert np.array_equal(flag.cpu().numpy(), fl)
    assert np.array_equal(idx.cpu().numpy(), want_i) and np.array_equal(cnt.cpu().numpy(), rc)
    assert np.array_equal(np.nan_to_num(sc.cpu().numpy(), nan=-7.0), np.nan_to_num(want_s, nan=-7.0))
    mlp.close()
    ctx.close()
