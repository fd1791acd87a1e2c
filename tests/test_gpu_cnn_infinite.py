"""An activation that overflows to infinity in training (GPU): the weight
gradients it is no term of stay finite.  The reductions run over whole MFMA
steps, whose places past the grid hold a zero gradient; an activation there must
not be infinite, since its product with that zero is NaN."""
import itertools

import numpy as np
import pytest

from paper_2508_05020_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,at", [(3, 8, (5, 5, 10)), (3, 8, (5, 5, 11)), (3, 8, (10, 11, 4)), (3, 8, (11, 11, 11)),
                                      (3, 8, (5, 5, 0)), (3, 8, (8, 0, 1)), (3, 8, (0, 0, 0)),
                                      (2, 8, (5, 11)), (2, 16, (19, 19)), (2, 10, (0, 0))])
def test_infinite_activation_reaches_its_own_terms_only(dim, n, at):
    import torch
    import paper_2508_05020_amd.amr as A
    ci, ch, cs = (4, 16, 4) if dim == 2 else (5, 8, 8)
    taps = list(itertools.product(range(3), repeat=dim))
    rng = np.random.default_rng(n)
    w1 = 0.1 * rng.normal(size=(ch, ci, len(taps)))
    w1[:, 0] = 0.0
    w1[0, 0, len(taps) // 2] = 4.0                 # the overflow: 4 times the largest BF16 number
    w2 = 0.1 * rng.normal(size=(ch, ch, len(taps)))
    w2[:, 0] = -0.1 - np.abs(w2[:, 0])             # -infinity behind it, which ReLU drops
    w3 = 0.1 * rng.normal(size=(ch, len(taps)))
    flat = np.concatenate([w1.ravel(), np.full(ch, 0.1), w2.ravel(), np.ones(ch), w3.ravel(), [0.0]])
    h = A.Hierarchy(W.AMRConfig(name="t", dim=dim, base_cells=32, patch_cells=[16], periodic=[True] * dim,
                                max_patches=64))
    net = A.Predictor(h, n, [0.0] * ci, [1.0] * ci, max_batch=1)
    net.set_weights(flat)
    x = np.zeros((n + 6,) * dim + (cs,), np.float32)
    x[..., :ci] = rng.normal(size=x.shape[:-1] + (ci,))
    x[..., 0] = 0.0
    x[tuple(c + 1 for c in at) + (0,)] = 3.3895314e38
    y = (rng.random(n ** dim) < 0.2).astype(np.uint8)
    xd = torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).cuda().reshape(1, -1, cs).contiguous()
    grads = torch.zeros(net.nparams, device="cuda")
    loss = net.train_step(xd, torch.from_numpy(y[None]).cuda(), lr=0.0, grads=grads).item()
    nan = np.zeros((ch, ch, len(taps)), bool)
    for k, tap in enumerate(taps):                 # a term of the sum: position at - tap of the grid
        nan[:, 0, k] = all(0 <= a - t < n + 2 for a, t in zip(at, tap))
    expected = np.concatenate([np.zeros(w1.size + ch, bool), nan.ravel(), np.zeros(ch + w3.size + 1, bool)])
    assert np.isfinite(loss)
    assert nan.any() and not nan[:, 0].all()
    assert np.array_equal(~np.isfinite(grads.cpu().numpy()), expected)
    net.close()
    h.close()
