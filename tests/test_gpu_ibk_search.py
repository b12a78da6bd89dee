"""The IBK search at the edges of its tiles and lists, against the FP64
oracle's exhaustive search.

Widths around the padded sizes (32, 64, 128, 256) and the 16-feature steps,
odd ones; every list length (k 1..16); databases of fewer samples than k, of
one tile, of a tile and one; queries of less and more than a workgroup's 256;
shares that are empty.  A nearly constant training column that the test
batch leaves (features of 10^4), which the FP32 features cannot certify; every
training kernel twice (equal distances).  Neighbour sets are exact, so
predictions match to the rounding of the output: 1e-5 (FP32) and 1e-9 (FP64)
on the speedup scale.
"""
import numpy as np
import pytest
import torch

from oracle import knn as N
from synthgen import make_batch

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(tr, te, D, E, k, f64, twice=False):
    from paper_1910_07776_amd import plain as G
    dt = torch.float64 if f64 else torch.float32
    ctx = G.Context(0)
    G.ibk_fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D, dt), dev(tr.counters), dev(tr.cycles), k=k)
    p = G.Plan(ctx, te.nopts, te.opt_ids, E, D, dt)
    _, grid = G.ibk_predict(ctx, p, dev(te.counters), dev(te.cycles), grid=True)
    n = G.ibk_exact_count(ctx, p)
    G.sync(ctx)
    want = N.predict_grid(N.database(tr, D), te, k, Bmax=p.Bmax)
    got = grid.cpu().numpy().astype(np.float64)
    pred = ~np.isnan(want)
    assert np.array_equal(~np.isnan(got), pred)
    err = np.abs(np.exp(got[pred]) - np.exp(want[pred])) / np.exp(want[pred])
    assert err.max(initial=0.0) <= (1e-9 if f64 else 1e-5), err.max()
    ctx.close()
    return n, int(pred.sum())


# events, double precision, k, optimisations, training kernels, test kernels
@pytest.mark.parametrize("E,f64,k,B,ktr,kte", [
    (1, False, 1, 3, 1, 1), (15, True, 4, 3, 2, 3), (16, False, 5, 5, 2, 9), (17, False, 10, 5, 1, 40),
    (32, True, 11, 5, 2, 33), (33, False, 16, 5, 3, 20), (64, False, 4, 4, 4, 65), (65, True, 10, 6, 1, 8),
    (128, False, 16, 6, 5, 12), (128, True, 5, 1, 33, 300), (129, False, 10, 4, 30, 16), (255, True, 16, 3, 40, 5),
    (256, False, 3, 6, 20, 9)])
def test_search_matches_the_oracle(E, f64, k, B, ktr, kte):
    npdt = np.float64 if f64 else np.float32
    tr = make_batch(400 + E, range(1000, 1000 + ktr), E, B, dtype=npdt)
    te = make_batch(400 + E, range(kte), E, B, dtype=npdt)
    check(tr, te, B, E, k, f64)


@pytest.mark.parametrize("E,k", [(40, 10), (128, 16)])
def test_features_far_from_the_training_set(E, k):
    tr = make_batch(11, range(1000, 1024), E, 5)
    te = make_batch(11, range(8), E, 5)
    r = np.random.default_rng(3)
    tr.counters[:, 1] = tr.cycles * (1.0 + 1e-4 * r.standard_normal(tr.N))
    te.counters[:, 1] = te.cycles * r.uniform(0.3, 3.0, te.N)
    n, queries = check(tr, te, 5, E, k, False)
    assert 0 < n <= queries   # FP32 features err by about 1e-2 there: searched again in FP64


def test_equal_distances():
    a = make_batch(12, list(range(1000, 1012)) * 2, 64, 4, dtype=np.float64)
    te = make_batch(12, list(range(1000, 1004)) + list(range(4)), 64, 4, dtype=np.float64)
    check(a, te, 4, 64, 7, True)
