"""A plan that has served short lists serves longer ones: the workspace of its
queries holds lists of any length, so the answers and flags of a query after
n_suggest (and the band's cap) was raised equal those of a new plan, with the
output layer's own ranking (64 and 128 subsets) and without."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K,raised", [(6, 300, (8, 64)), (6, 300, (8, 4)), (7, 65, (5, 4)), (8, 20, (8, 64))])
def test_longer_lists_after_a_short_query(B, K, raised):
    from paper_1910_07776_amd import plain as G, surrogate as S
    from synthgen import make_batch
    E, D = 40, 8
    ctx = G.Context(0, n_suggest=3, tau=0.02)
    tr = make_batch(17, range(64), E, D)
    G.fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D), torch.from_numpy(tr.counters).cuda(),
          torch.from_numpy(tr.cycles).cuda())
    te = make_batch(17, range(500, 500 + K), E, D, brange=(B, B))
    c, cy = torch.from_numpy(te.counters).cuda(), torch.from_numpy(te.cycles).cuda()
    mlp = S.MLP(ctx, E, 512, 1 << B, max_batch=K, seed=18)
    mlp.unflatten(mlp.params)["b3"].copy_(torch.linspace(-0.2, 0.1, 1 << B))
    mlp.freeze()

    def query(plan, n, cap):
        out = {"idx": torch.full((K, n), -9, dtype=torch.int32, device="cuda"),
               "score": torch.full((K, n), -9.0, device="cuda"),
               "count": torch.full((K,), -9, dtype=torch.int32, device="cuda")}
        flag = torch.full((K,), -9, dtype=torch.int32, device="cuda")
        G.serve_query(ctx, plan, mlp, c, cy, out, flag, tol=9.0, band=0.05, cap=cap)
        G.sync(ctx)
        return [np.nan_to_num(t.cpu().numpy(), nan=-7.0) for t in (*out.values(), flag)]

    served = G.Plan(ctx, te.nopts, te.opt_ids, E, D)
    query(served, 3, 4)
    n, cap = raised
    ctx.set_params(n_suggest=n)
    got = query(served, n, cap)
    want = query(G.Plan(ctx, te.nopts, te.opt_ids, E, D), n, cap)
    for g, w in zip(got, want):
        assert np.array_equal(g, w)
    assert (got[2] > 3).any()
    mlp.close()
    ctx.close()
