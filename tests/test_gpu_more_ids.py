"""A plan that names more global ids than the model was trained on, its kernels
having none of the further ones: nearest neighbours, model trees and the linear
models give what a plan of the model's own ids gives."""
import numpy as np
import pytest
import torch

from synthgen import make_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more", [1, 58])
def test_plan_of_more_ids_than_the_model(more):
    from paper_1910_07776_amd import plain as G
    E, D = 40, 6
    ctx = G.Context(0)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tr, te = make_batch(61, range(100, 130), E, D), make_batch(61, range(20), E, D)
    train = G.Plan(ctx, tr.nopts, tr.opt_ids, E, D)
    for f in (G.fit, G.ibk_fit, G.m5p_fit):
        f(ctx, train, dev(tr.counters), dev(tr.cycles))
    c, cy = dev(te.counters), dev(te.cycles)
    outs = []
    for ids in (D, D + more):
        p = G.Plan(ctx, te.nopts, te.opt_ids, E, ids)
        outs.append([t for f in (G.predict, G.ibk_predict, G.m5p_predict) for t in f(ctx, p, c, cy, grid=True)])
    G.sync(ctx)
    for a, b in zip(*outs):
        assert torch.equal(torch.nan_to_num(a, nan=7e7), torch.nan_to_num(b, nan=7e7))
    ctx.close()
