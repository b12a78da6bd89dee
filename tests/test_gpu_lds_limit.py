"""The streaming form at the limit of a workgroup's LDS: kernels of 1024, 512, 16
and 8 versions in one chunk beside the FP64 weights of 64 optimisations and 256
events take 163,824 of the 163,840 bytes.  The pass, its grid and its masked
form run and equal the fused form, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_chunk_as_large_as_the_lds():
    from paper_1910_07776_amd import plain as G
    E, D, B = 256, 64, np.array([10, 9, 4, 3], np.int32)
    rng = np.random.default_rng(3)
    ctx = G.Context(0, tau=-1.0)
    ctx.model_set({"mu": rng.normal(0, 0.1, E), "sigma": rng.uniform(0.5, 1.5, E),
                   "W": rng.normal(0, 0.02, (D, E + 1)), "counts": np.full(D, 9)})
    ids = np.concatenate([np.sort(rng.choice(D, b, replace=False)) for b in B]).astype(np.int32)
    new, ref = (G.Plan(ctx, B, ids, E, D, torch.float64) for _ in range(2))
    new.set_items(int(new.N))
    new.set_launch(4, -2, 0)
    ref.set_launch(4, 1, 0)
    c = torch.from_numpy(np.exp(rng.normal(0, 0.3, (new.N, E)))).cuda()
    cy = torch.from_numpy(np.exp(rng.normal(0, 0.3, new.N))).cuda()
    got, want = ([*G.suggest(ctx, p, c, cy), *G.predict(ctx, p, c, cy, grid=True)] for p in (new, ref))
    for p, o in ((new, got), (ref, want)):
        sub = {"idx": torch.zeros_like(o[0]), "score": torch.zeros_like(o[1]), "count": torch.zeros_like(o[2]),
               "table": torch.zeros_like(o[3])}
        G.suggest_subset(ctx, p, c, cy, torch.tensor([0, 1, 0, 1], dtype=torch.int32, device="cuda"), sub)
        o.extend(sub.values())
    G.sync(ctx)
    for a, b in zip(got, want):
        assert torch.equal(torch.nan_to_num(a, nan=7e7), torch.nan_to_num(b, nan=7e7))
    ctx.close()
