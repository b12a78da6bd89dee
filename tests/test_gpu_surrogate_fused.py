"""Frozen inference in one launch (batches of 8192 and more, and the call that
forms the features and ranks at any size) against the layer-by-layer forward
of the same parameters: both form every sum in the same order, so outputs and
lists are compared bit for bit."""
import numpy as np
import pytest
import torch

from paper_1910_07776_amd._abi import SuggError

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    from paper_1910_07776_amd import plain, surrogate
    c = plain.Context(0)
    yield plain, surrogate, c
    c.close()


def fused(mlp):
    """Whether the last call reported the one-launch instance: the same
    instance for all three layers (64-row tiles of 512 hidden units)."""
    import ctypes as C
    from paper_1910_07776_amd import _abi as A
    info = np.zeros(32, np.int32)
    assert A.lib().sugg_mlp_launch_info(mlp.h, info.ctypes.data_as(A._PI32)) == 0
    return info.reshape(8, 4)[:3].tolist()


def same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


def lists_equal(plain, ctx, y, got, n, tau):
    B, out = y.shape
    seg = torch.arange(0, B + 1, dtype=torch.int64, device="cuda") * out
    ri, rs, rc = plain.rank_suggest(ctx, y.reshape(-1), seg, n=n, tau=tau, skip_head=1)
    plain.sync(ctx)
    idx, sc, cnt = got
    assert torch.equal(idx, ri) and torch.equal(cnt, rc)
    assert torch.equal(torch.nan_to_num(sc, nan=-7.0), torch.nan_to_num(rs, nan=-7.0))


@pytest.mark.parametrize("n_in,out,B", [
    (8, 32, 8192), (40, 64, 8193), (128, 96, 8255), (128, 128, 8256), (264, 256, 8200), (512, 512, 8192),
    (136, 544, 8211), (128, 1024, 9001), (128, 64, 16385)])
def test_one_launch_equals_layer_by_layer(S, n_in, out, B):
    plain, sur, ctx = S
    mlp = sur.MLP(ctx, n_in, 512, out, max_batch=B, seed=51)
    mlp.freeze()
    g = torch.Generator(device="cuda").manual_seed(52)
    x = torch.randn(B, n_in, device="cuda", generator=g)
    x[1] = 0.0
    x[-1] *= 300.0
    x[2, 0] = float("nan")      # a row's NaN and infinity stay in that row
    x[3, n_in - 1] = float("inf")
    y = mlp.infer(x)
    plain.sync(ctx)
    info = fused(mlp)
    assert info[0] == info[1] and info[0][0] == 64, info
    y0 = mlp(x)
    plain.sync(ctx)
    ok = ~torch.isnan(y0)
    assert torch.equal(torch.isnan(y), ~ok) and same(y[ok], y0[ok]) and bool(ok[4:].all())
    # an output that is not aligned to 16 bytes takes the layers one by one
    buf = torch.empty(B * out + 1, device="cuda")
    yu = mlp.infer(x, y=buf[1:].view(B, out))
    plain.sync(ctx)
    assert same(yu[ok], y0[ok])
    x[2:4] = 1.0
    for n, tau in ((3, 0.02), (8, -0.01)):
        y2 = torch.empty(B, out, device="cuda")
        got = mlp.infer_rank(x, n=n, tau=tau, skip=1, y=y2)
        lists_equal(plain, ctx, mlp(x), got, n, tau)
        assert same(y2, mlp(x))
    # other parameters frozen again: the operand-order copy follows
    p2 = mlp.params * 0.5
    mlp.freeze(p2)
    assert same(mlp.infer(x), mlp.forward_raw(p2, x))
    mlp.close()


@pytest.mark.parametrize("K,E,out,n", [(1, 128, 64, 3), (63, 40, 64, 8), (65, 128, 128, 3), (1000, 8, 64, 1),
                                       (8200, 128, 256, 3)])
def test_features_and_network_in_one_launch(S, K, E, out, n):
    plain, sur, _ = S
    ctx = plain.Context(0, n_suggest=n)
    from synthgen import make_batch
    D = out.bit_length() - 1
    tr = make_batch(43, range(100, 164), E, D)
    plain.fit(ctx, plain.Plan(ctx, tr.nopts, tr.opt_ids, E, D), torch.from_numpy(tr.counters).cuda(),
              torch.from_numpy(tr.cycles).cuda())
    p = plain.Plan(ctx, np.full(K, D, np.int32), np.tile(np.arange(D, dtype=np.int32), K), E, D)
    g = torch.Generator(device="cuda").manual_seed(44)
    c = torch.empty(K << D, E, device="cuda").uniform_(1.0, 1e6, generator=g)
    cy = torch.empty(K << D, device="cuda").uniform_(1e5, 1e7, generator=g)
    mlp = sur.MLP(ctx, E, 512, out, max_batch=K, seed=45)
    mlp.freeze()
    idx, sc, cnt, table = plain.surrogate_suggest(ctx, p, mlp, c, cy, table=True)
    zz = plain.load_features(ctx, p, c, cy, baseline=True)
    y = mlp(zz)
    assert same(table, y)
    lists_equal(plain, ctx, y, (idx, sc, cnt), n, plain.TAU)
    c[(K - 1) << D, E - 1] = 0.0     # a counter that is not positive is reported
    plain.surrogate_suggest(ctx, p, mlp, c, cy)
    with pytest.raises(SuggError):
        plain.sync(ctx)
    mlp.close()
    ctx.close()
