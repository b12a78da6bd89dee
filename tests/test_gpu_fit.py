"""The ridge fit's kernels at the edges of their tiles, against the FP64 oracle.

Widths around the 16-column blocks and the three instances (64, 128, 256
events), odd widths (no vector loads), solves in LDS and in global memory
(from 175 events), few rows (one pair list per optimisation) and many (rows
grouped by the set of optimisations they are before versions of), optimisations
without a pair, stages that are not full.

What is compared is the residual of the oracle's normal equations,
|A w - r| <= 1e-11 (|A| |w| + |r|) (Frobenius and 2-norms): sums of at most
2^13 products carry 2^13 eps = 1.8e-12, the features 1e-12 (four units in the
last place of a log of size 10, over a standard deviation of at least 0.02),
the factorisation 257 eps; their sum stays below 1e-11.
"""
import numpy as np
import pytest
import torch

from oracle import plain as P
from synthgen import make_batch

pytestmark = pytest.mark.gpu

# events, double precision, ids, optimisations per kernel, kernels
CASES = [(1, True, 3, (3, 3), 5), (15, False, 4, (4, 4), 40), (16, False, 6, (6, 6), 3), (17, True, 6, (6, 6), 64),
         (40, True, 6, (6, 6), 2), (64, False, 10, (4, 10), 20), (65, False, 6, (0, 6), 33), (100, False, 10, (4, 8), 300),
         (126, False, 12, (1, 3), 50), (127, True, 6, (6, 6), 64), (128, False, 6, (6, 6), 129),
         (128, False, 40, (2, 9), 60), (129, False, 6, (5, 5), 100), (174, False, 5, (5, 5), 90),
         (175, True, 5, (5, 5), 90), (256, False, 10, (4, 9), 70), (255, False, 64, (3, 7), 80)]


@pytest.mark.parametrize("E,f64,D,brange,K", CASES)
def test_fit_solves_the_normal_equations(E, f64, D, brange, K):
    from paper_1910_07776_amd import plain as G
    b = make_batch(77 + E, range(K), E, D, brange=brange, dtype=np.float64 if f64 else np.float32)
    ctx = G.Context(0)
    p = G.Plan(ctx, b.nopts, b.opt_ids, E, D, torch.float64 if f64 else torch.float32)
    c, cyc = torch.from_numpy(b.counters).cuda(), torch.from_numpy(b.cycles).cuda()
    for _ in range(2):   # the second fit reuses the plan's workspace
        G.fit(ctx, p, c, cyc)
        G.sync(ctx)
        m = ctx.model_get()
        x = P.features(b.counters, b.cycles)
        mu, sg = P.column_stats(x)
        assert np.allclose(m["mu"], mu, rtol=0, atol=1e-12) and np.allclose(m["sigma"], sg, rtol=1e-11, atol=0)
        z = P.standardize(x, mu, sg)
        opt, before, after, *_ = P.candidate_pairs(b.nopts, b.opt_ids, b.opt_off, b.row_off)
        y = P.pair_labels(b.cycles, before, after)
        for o in range(D):
            q = opt == o
            assert m["counts"][o] == q.sum()
            if not q.any():
                assert np.isnan(m["W"][o]).all()
                continue
            X = np.concatenate([z[before[q]], np.ones((int(q.sum()), 1))], axis=1)
            A = X.T @ X + np.diag([P.LAMBDA] * E + [0.0])
            r = X.T @ y[q]
            w = m["W"][o]
            err = np.linalg.norm(A @ w - r)
            bound = 1e-11 * (np.linalg.norm(A) * np.linalg.norm(w) + np.linalg.norm(r))
            assert err <= bound, (o, err, bound)
    ctx.close()
