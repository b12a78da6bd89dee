"""A bad counter anywhere in a batch scored by model trees is reported: in every
lane's columns of a row (the first, one in the middle, the last), in versions
that predictions start from and in those that none starts from, in the
one-launch pass, the tiled pass and the grid."""
import numpy as np
import pytest
import torch

from paper_1910_07776_amd._abi import SuggError
from synthgen import make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,f64,brange", [(128, False, (6, 6)), (37, False, (4, 5)), (200, False, (7, 7)),
                                          (64, True, (1, 4)), (128, False, (8, 9)), (37, True, (8, 8)),
                                          (256, True, (8, 8))])
def test_every_column_is_checked(E, f64, brange):
    from paper_1910_07776_amd import plain as G
    dt, nd = (torch.float64, np.float64) if f64 else (torch.float32, np.float32)
    ctx = G.Context(0)
    D = 9
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tr = make_batch(51, range(500, 540), E, D, brange=(3, 6), dtype=nd)
    G.m5p_fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D, dt), dev(tr.counters), dev(tr.cycles))
    te = make_batch(52, range(5), E, D, brange=brange, dtype=nd)
    p = G.Plan(ctx, te.nopts, te.opt_ids, E, D, dt)
    c, cy = dev(te.counters), dev(te.cycles)
    passes = (lambda: G.m5p_suggest(ctx, p, c, cy), lambda: G.m5p_predict(ctx, p, c, cy, grid=True))
    last = int(te.row_off[1]) - 1            # a version no prediction starts from
    for row in (0, 1, last, p.N - 2):
        for col in (0, 5, E // 2, E - 1):
            keep = c[row, col].clone()
            for v in (0.0, -1.0, float("nan"), float("inf")):
                c[row, col] = v
                for f in passes:
                    f()
                    with pytest.raises(SuggError) as e:
                        G.sync(ctx)
                    assert e.value.name == "SUGG_E_BAD_COUNTER"
            c[row, col] = keep
    for f in passes:
        f()
    G.sync(ctx)
    ctx.close()
