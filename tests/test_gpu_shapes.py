"""Launch shapes a new plan can get, against the fused kernel set explicitly.

A new plan's scoring pass takes the streaming or the fused form by its rows,
its largest kernel and the width, with wide workgroups where its chunks are
large and few; the grid and the masked pass follow it.  Tables, grids and lists
must equal the fused form's (4 waves, one row per stage) bit for bit, on both
sides of each line of that rule: kernels of 1 to 4096 versions, one chunk and
many, odd widths, both types, lists of 3 and 8.  The all-paths table (whose
wide workgroups start at 256 versions) is compared with the oracle to 1e-5
(FP32) and 1e-9 (FP64) on the speedup scale.
"""
import numpy as np
import pytest
import torch

from oracle import paths as Q
from oracle import plain as P
from synthgen import make_batch

pytestmark = pytest.mark.gpu

# events, double precision, ids, optimisations per kernel, kernels, list length
CASES = [(1, False, 3, (0, 3), 9, 3), (40, True, 6, (6, 6), 2, 3), (64, False, 7, (7, 7), 3, 8), (65, True, 8, (7, 8), 5, 3),
         (128, False, 6, (6, 6), 700, 3), (128, False, 10, (10, 10), 3, 8), (100, False, 10, (9, 10), 40, 3),
         (101, False, 10, (4, 9), 300, 3), (256, False, 9, (9, 9), 7, 3), (200, True, 10, (8, 10), 12, 8),
         (33, False, 12, (12, 12), 2, 3), (128, False, 9, (9, 9), 1000, 3), (16, True, 11, (5, 11), 60, 8),
         (128, False, 6, (4, 6), 1900, 3), (40, False, 6, (6, 6), 4150, 3), (150, False, 6, (5, 6), 2900, 3)]


def setup(E, f64, D, brange, K, n):
    from paper_1910_07776_amd import plain as G
    dt = torch.float64 if f64 else torch.float32
    tr = make_batch(900 + E, range(5000, 5048), E, D, brange=(min(4, D), min(6, D)), dtype=np.float64 if f64 else np.float32)
    te = make_batch(900 + E, range(K), E, D, brange=brange, dtype=np.float64 if f64 else np.float32)
    ctx = G.Context(0, n_suggest=n)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    G.fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D, dt), dev(tr.counters), dev(tr.cycles))
    G.sync(ctx)
    return G, ctx, te, dt, dev(te.counters), dev(te.cycles)


def same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=7e7), torch.nan_to_num(b, nan=7e7))


@pytest.mark.parametrize("E,f64,D,brange,K,n", CASES)
def test_a_new_plans_shape_gives_the_fused_forms_results(E, f64, D, brange, K, n):
    G, ctx, te, dt, c, cy = setup(E, f64, D, brange, K, n)
    new = G.Plan(ctx, te.nopts, te.opt_ids, E, D, dt)
    ref = G.Plan(ctx, te.nopts, te.opt_ids, E, D, dt)
    ref.set_launch(4, 1, 0)
    want, got = G.suggest(ctx, ref, c, cy), G.suggest(ctx, new, c, cy)
    for w, g in zip(want, got):
        assert same(w, g)
    tw, gw = G.predict(ctx, ref, c, cy, grid=True)
    tg, gg = G.predict(ctx, new, c, cy, grid=True)
    assert same(tw, tg) and same(gw, gg) and same(tg, got[3])
    mask = torch.from_numpy((np.random.default_rng(E).random(K) < 0.3).astype(np.int32)).cuda()
    outs = []
    for p in (ref, new):
        o = {"idx": torch.full((K, n), -7, dtype=torch.int32, device="cuda"),
             "score": torch.full((K, n), -7.0, dtype=dt, device="cuda"),
             "count": torch.full((K,), -7, dtype=torch.int32, device="cuda"),
             "table": torch.full((p.N,), -7.0, dtype=dt, device="cuda")}
        G.suggest_subset(ctx, p, c, cy, mask, o)
        outs.append(o)
    for k in outs[0]:
        assert same(outs[0][k], outs[1][k])
    sel = mask.bool()
    assert same(outs[1]["score"][sel], want[1][sel]) and bool((outs[1]["count"][~sel] == -7).all())
    G.sync(ctx)
    ctx.close()


@pytest.mark.parametrize("E,f64,D,brange,K,n", [c for c in CASES if c[3][1] <= 10])
def test_allpaths_matches_the_oracle(E, f64, D, brange, K, n):
    K = min(K, 20)
    G, ctx, te, dt, c, cy = setup(E, f64, D, brange, K, n)
    table, idx, score, count = G.predict_allpaths(ctx, G.Plan(ctx, te.nopts, te.opt_ids, E, D, dt), c, cy)
    G.sync(ctx)
    m = ctx.model_get()
    grid = P.predict_grid({"mu": m["mu"], "sigma": m["sigma"], "W": m["W"]}, te)
    want = Q.compose_allpaths(grid, te)
    got = table.cpu().numpy().astype(np.float64)
    rtol = 1e-9 if f64 else 1e-5
    assert (np.abs(np.exp(got) - np.exp(want)) <= rtol * np.exp(want)).all()
    # the lists are the table's own top n, exactly
    for k in range(K):
        seg = table[int(te.row_off[k]):int(te.row_off[k + 1])]
        v, s = seg.cpu().numpy(), np.arange(len(seg))
        keep = s[(s > 0) & (v > seg.new_tensor(ctx.params["tau"]).item())]
        top = keep[np.lexsort((keep, -v[keep]))][:n]
        assert int(count[k]) == len(top) and idx[k, :len(top)].tolist() == top.tolist()
        assert score[k, :len(top)].cpu().numpy().tolist() == v[top].tolist()
    ctx.close()


@pytest.mark.parametrize("E,f64,brange,K", [(16, False, (6, 6), 8200), (20, False, (0, 4), 20001), (128, False, (10, 10), 130),
                                            (40, True, (5, 9), 400), (33, False, (8, 8), 65)])
def test_masked_pass_takes_exactly_the_selected_kernels(E, f64, brange, K):
    """Masks of no kernel, one, the last, a third, whole stretches of 64
    chunks and all: the selected kernels' outputs are the whole pass's bit for
    bit, the others' stay as they were (chunks of one and of many kernels)."""
    n, D = 3, 10
    G, ctx, _, dt, _, _ = setup(E, f64, D, (4, 4), 1, n)
    rng = np.random.default_rng(K)
    B = rng.integers(brange[0], brange[1] + 1, K).astype(np.int32)
    ids = np.concatenate([np.sort(rng.choice(D, b, replace=False)) for b in B]).astype(np.int32)
    p = G.Plan(ctx, B, ids, E, D, dt)
    g = torch.Generator(device="cuda").manual_seed(5)
    c = torch.empty(p.N, E, dtype=dt, device="cuda").uniform_(1.0, 1e5, generator=g)
    cy = torch.empty(p.N, dtype=dt, device="cuda").uniform_(1e5, 1e6, generator=g)
    full = G.suggest(ctx, p, c, cy)
    rowk = torch.from_numpy(np.repeat(np.arange(K), 1 << B.astype(np.int64))).cuda()
    third = (rng.random(K) < 0.3).astype(np.int32)
    stretch = ((np.arange(K) // 64) % 2).astype(np.int32)
    for m in (np.zeros(K), np.eye(1, K, K // 2)[0], np.eye(1, K, K - 1)[0], third, stretch, np.ones(K)):
        mask = torch.from_numpy(m.astype(np.int32)).cuda()
        o = {"idx": torch.full((K, n), -7, dtype=torch.int32, device="cuda"),
             "score": torch.full((K, n), -7.0, dtype=dt, device="cuda"),
             "count": torch.full((K,), -7, dtype=torch.int32, device="cuda"),
             "table": torch.full((p.N,), -7.0, dtype=dt, device="cuda")}
        G.suggest_subset(ctx, p, c, cy, mask, o)
        for got, want, sel in zip((o["idx"], o["score"], o["count"], o["table"]), full,
                                  (mask.bool(),) * 3 + (mask.bool()[rowk],)):
            s = sel.view(-1, *([1] * (got.dim() - 1)))
            assert same(got, torch.where(s, want, torch.full_like(want, -7)))
    G.sync(ctx)
    ctx.close()
