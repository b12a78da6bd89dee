"""The one-launch model-tree pass (kernels of at most 128 versions) against the
tiled form, which the grid output takes: the composed tables must be equal bit
for bit, the lists those of the ranking call on the table (FP64 plans), for
every workgroup size, mixed batches and odd widths; and a bad counter in a
version no prediction starts from is still reported."""
import numpy as np
import pytest
import torch

from paper_1910_07776_amd._abi import SuggError
from synthgen import make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,f64,brange,n", [(128, False, (4, 4), 3), (40, True, (5, 5), 8), (37, False, (0, 5), 3),
                                            (128, True, (6, 6), 8), (200, False, (7, 7), 3), (128, True, (7, 7), 3),
                                            (65, True, (0, 7), 8), (1, True, (1, 7), 3), (40, True, (2, 9), 3),
                                            (256, True, (0, 3), 8)])
def test_forms_agree(E, f64, brange, n):
    from paper_1910_07776_amd import plain as G
    dt, nd = (torch.float64, np.float64) if f64 else (torch.float32, np.float32)
    ctx = G.Context(0, n_suggest=n)
    D = 9
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tr = make_batch(51, range(500, 540), E, D, brange=(3, 6), dtype=nd)
    G.m5p_fit(ctx, G.Plan(ctx, tr.nopts, tr.opt_ids, E, D, dt), dev(tr.counters), dev(tr.cycles))
    te = make_batch(51, range(37), E, D, brange=brange, dtype=nd)
    p = G.Plan(ctx, te.nopts, te.opt_ids, E, D, dt)
    c, cy = dev(te.counters), dev(te.cycles)
    table_g, _ = G.m5p_predict(ctx, p, c, cy, grid=True)
    table_e, _ = G.m5p_predict(ctx, p, c, cy)
    idx, score, count, table = G.m5p_suggest(ctx, p, c, cy)
    G.sync(ctx)
    assert torch.equal(table_g, table_e) and torch.equal(table_e, table)
    seg = torch.from_numpy(np.asarray(te.row_off, np.int64)).cuda()
    ri, rs, rc = G.rank_suggest(ctx, table.view(-1), seg, n=n, tau=G.TAU, skip_head=1)
    G.sync(ctx)
    assert torch.equal(count, rc)
    if f64:
        assert torch.equal(idx, ri)
        assert torch.equal(torch.nan_to_num(score, nan=-7.0), torch.nan_to_num(rs, nan=-7.0))
    for row in {0, p.N // 2, p.N - 1}:
        for t, at in ((c, (row, 0)), (cy, (row,))):
            keep = t[at].clone()
            for v in (0.0, -1.0, float("nan"), float("inf")):
                t[at] = v
                G.m5p_suggest(ctx, p, c, cy)
                with pytest.raises(SuggError):
                    G.sync(ctx)
            t[at] = keep
    G.m5p_suggest(ctx, p, c, cy)
    G.sync(ctx)
    ctx.close()
