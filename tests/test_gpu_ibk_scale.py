"""The IBK search where one training version sets the scale of the stored
halves: its counters are e^600 times the others', so the others' features are
small beside the largest stored value and the lower halves of many lie below
FP16's normal range.  The neighbours must still be the exact ones: predictions
match the FP64 oracle's to the rounding of the output, 1e-9 on the speedup
scale, also for queries that are stored vectors themselves."""
import numpy as np
import pytest
import torch

from oracle import knn as N
from synthgen import make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,columns", [(16, 3, 16), (40, 10, 40), (100, 16, 50)])
def test_a_version_far_from_all_others(E, k, columns):
    from paper_1910_07776_amd import plain as G
    D = 6
    tr = make_batch(21, range(1000, 1048), E, D, dtype=np.float64)
    te = make_batch(21, list(range(6)) + [1003, 1040], E, D, dtype=np.float64)   # the last two are training kernels
    tr.counters[tr.N // 2 + 5, :columns] *= np.exp(600.0)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = G.Context(0)
    G.ibk_fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D, torch.float64), dev(tr.counters), dev(tr.cycles), k=k)
    p = G.Plan(ctx, te.nopts, te.opt_ids, E, D, torch.float64)
    _, grid = G.ibk_predict(ctx, p, dev(te.counters), dev(te.cycles), grid=True)
    G.sync(ctx)
    want = N.predict_grid(N.database(tr, D), te, k, Bmax=p.Bmax)
    got = grid.cpu().numpy()
    pred = ~np.isnan(want)
    assert np.array_equal(~np.isnan(got), pred)
    assert (np.abs(np.exp(got[pred]) - np.exp(want[pred])) <= 1e-9 * np.exp(want[pred])).all()
    ctx.close()
