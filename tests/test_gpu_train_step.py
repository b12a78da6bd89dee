"""An epoch in one call (output layer and the backward through it in one
launch, gradients, Adam and the next gather in one) against the separate step
on the gathered batches: parameters, moments, gradients and losses bit for bit,
at batches of whole and partial tiles and output widths on both sides of the
one-launch output layer."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,batch", [((128, 512, 64), 4096), ((128, 512, 64), 1), ((40, 512, 64), 33),
                                        ((128, 512, 128), 320), ((128, 512, 128), 97), ((8, 512, 64), 1000),
                                        ((128, 512, 64), 2112), ((128, 512, 256), 200), ((128, 256, 64), 130)])
def test_epoch_equals_steps(dims, batch):
    from paper_1910_07776_amd import plain, surrogate as sur
    ctx = plain.Context(0)
    i, h, o = dims
    n, steps = 3 * batch + 7, 3
    rng = np.random.default_rng(batch)
    X = torch.tensor(rng.normal(size=(n, i)), dtype=torch.float32, device="cuda")
    Y = torch.tensor(rng.normal(size=(n, o)) * 0.2, dtype=torch.float32, device="cuda")
    perm = torch.tensor(rng.permutation(n)[:steps * batch], dtype=torch.int32, device="cuda")
    a = sur.MLP(ctx, i, h, o, max_batch=batch, seed=4)
    b = sur.MLP(ctx, i, h, o, max_batch=batch, seed=4)
    la = a.train_epoch(X, Y, perm, batch, lr=2e-3)
    lb = []
    for s in range(steps):
        idx = perm[s * batch:(s + 1) * batch].long()
        lb.append(b.train_step(X[idx].contiguous(), Y[idx].contiguous(), lr=2e-3).clone())
    plain.sync(ctx)
    assert torch.equal(la, torch.cat(lb))
    assert torch.equal(a.grads, b.grads)
    assert torch.equal(a.params, b.params) and torch.equal(a.m, b.m) and torch.equal(a.v, b.v)
    # what the last step kept serves a backward of its own: the output layer's
    # gradients are the step's (the others pass through the updated weights)
    g, want = a.backward_raw(a.params, None, batch, torch.empty_like(a.params)), a.grads
    plain.sync(ctx)
    for name in ("W3", "b3"):
        assert torch.equal(a.unflatten(g)[name], a.unflatten(want)[name])
    a.close()
    b.close()
    ctx.close()
