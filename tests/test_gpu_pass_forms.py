"""The form each pass of a plan takes by itself (its rows, its kernels' sizes,
the model's size, the lists' length) against the fused kernel set explicitly:
tables, grids, lists and masked passes equal bit for bit, for batches of very
small kernels, on both sides of the lines by mean size and by rows, beside a
model of 64 KB, and for lists that were made longer after the plan."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# events, double precision, ids, optimisations per kernel, rows, list length (before, after)
CASES = [(40, False, 10, (0, 0), 70000, (3, 3)), (64, False, 10, (0, 2), 300000, (3, 3)),
         (130, False, 10, (1, 3), 70000, (3, 8)), (33, True, 10, (2, 2), 70000, (3, 3)),
         (129, False, 10, (3, 3), 100000, (3, 3)), (129, False, 10, (3, 3), 270000, (3, 3)),
         (64, True, 10, (2, 4), 300000, (8, 3)), (20, False, 10, (4, 4), 330000, (3, 8)),
         (20, False, 10, (4, 4), 1600000, (3, 3)), (16, False, 10, (4, 6), 1600000, (3, 8)),
         (256, False, 64, (4, 6), 70000, (3, 3)), (256, False, 64, (7, 7), 530000, (3, 3)),
         (200, True, 40, (5, 6), 70000, (3, 3)), (128, True, 64, (6, 6), 70000, (3, 3)),
         (40, False, 10, (0, 9), 3000, (3, 3))]


@pytest.mark.parametrize("E,f64,D,brange,rows,n", CASES)
def test_forms_agree(E, f64, D, brange, rows, n):
    from paper_1910_07776_amd import plain as G
    dt = torch.float64 if f64 else torch.float32
    rng = np.random.default_rng(rows + E)
    sizes = np.arange(brange[0], brange[1] + 1)
    K = int(rows / (2.0 ** sizes).mean()) + 1
    B = rng.choice(sizes, K).astype(np.int32)
    if brange == (0, 9):
        B[:] = 0
        B[K // 3] = 9                        # one large kernel among single versions
    has = np.argsort(np.argsort(rng.random((K, D)), axis=1), axis=1) < B[:, None]
    ids = np.nonzero(has)[1].astype(np.int32)
    ctx = G.Context(0, n_suggest=n[0], tau=-0.05)
    ctx.model_set({"mu": rng.normal(0, 0.1, E), "sigma": rng.uniform(0.5, 1.5, E),
                   "W": rng.normal(0, 0.02, (D, E + 1)), "counts": np.full(D, 9)})
    new, ref = (G.Plan(ctx, B, ids, E, D, dt) for _ in range(2))
    ref.set_launch(4, 1, 0)
    ctx.set_params(n_suggest=n[1])
    g = torch.Generator(device="cuda").manual_seed(E)
    c = torch.randn(new.N, E, generator=g, device="cuda", dtype=dt).mul_(0.3).exp_()
    cy = torch.randn(new.N, generator=g, device="cuda", dtype=dt).mul_(0.3).exp_()
    mask = torch.from_numpy((rng.random(K) < 0.3).astype(np.int32)).cuda()
    outs = []
    for p in (new, ref):
        o = [*G.suggest(ctx, p, c, cy), G.predict(ctx, p, c, cy)[0], *G.predict(ctx, p, c, cy, grid=True)]
        s = {"idx": torch.full((K, n[1]), -7, dtype=torch.int32, device="cuda"),
             "score": torch.full((K, n[1]), -7.0, dtype=dt, device="cuda"),
             "count": torch.full((K,), -7, dtype=torch.int32, device="cuda"),
             "table": torch.full((p.N,), -7.0, dtype=dt, device="cuda")}
        G.suggest_subset(ctx, p, c, cy, mask, s)
        outs.append(o + list(s.values()))
    G.sync(ctx)
    for a, b in zip(*outs):
        assert torch.equal(torch.nan_to_num(a, nan=7e7), torch.nan_to_num(b, nan=7e7))
    ctx.close()
