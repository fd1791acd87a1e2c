"""The fused training launch at the edges of its range (GPU): the smallest and
largest 2D patch edges, edges whose pixel counts are no multiple of an MFMA
row block, single tiles and batches that do not divide the waves, against an
FP64 backward through the oracle's layers at the activations that the network
has (weights and activations rounded to BF16; a ReLU mask that a rounding
flips would otherwise count as an error of the gradient).

Tolerance: what is left are the roundings of the activations that an
accumulation order moves and of the two layer gradients (2^-9 each): three
meet in a gradient at most, 3 * 2^-9 = 6e-3 relative in the L2 norm, taken
three times over for the loss's weighting of few positive cells.
"""
import numpy as np
import pytest

from oracle import cnn
from paper_2508_05020_amd import workloads as W

pytestmark = pytest.mark.gpu


def _params(flat, dim):
    ci, ch, k = (4, 16, (3, 3)) if dim == 2 else (5, 8, (3, 3, 3))
    shapes = [(ch, ci) + k, (ch,), (ch, ch) + k, (ch,), (1, ch) + k, (1,)]
    out, at = [], 0
    for s in shapes:
        size = int(np.prod(s))
        out.append(np.asarray(flat[at:at + size], np.float64).reshape(s))
        at += size
    return out


@pytest.mark.parametrize("dim,n,tiles", [(2, 8, 1), (2, 10, 3), (2, 16, 17), (2, 22, 5), (2, 32, 2),
                                         (3, 8, 1), (3, 8, 17)])
def test_training_gradients(dim, n, tiles):
    import torch
    import paper_2508_05020_amd.amr as A
    cfg = W.AMRConfig(name="t", dim=dim, base_cells=32, patch_cells=[16], periodic=[True] * dim,
                      max_patches=64)
    h = A.Hierarchy(cfg)
    ci, cs = (4, 4) if dim == 2 else (5, 8)
    net = A.Predictor(h, n, [0.0] * ci, [1.0] * ci, pos_weight=4.0, max_batch=tiles)
    rng = np.random.default_rng(100 * n + tiles)
    params = cnn.init_params(ci, 16 if dim == 2 else 8, dim, seed=n)
    net.set_weights(np.concatenate([(p + 0.05 * rng.normal(size=np.shape(p))).ravel() for p in params]))
    shape = (tiles,) + (n + 6,) * dim
    x = np.zeros(shape + (cs,), np.float32)
    x[..., :ci] = cnn.bf16_round(rng.normal(size=shape + (ci,)))
    y = (rng.random((tiles, n ** dim)) < 0.2).astype(np.uint8)
    xd = torch.from_numpy(x).to(torch.bfloat16).view(torch.int16).cuda().reshape(tiles, -1, cs).contiguous()
    grads = torch.zeros(net.nparams, device="cuda")
    loss = net.train_step(xd, torch.from_numpy(y).cuda(), lr=0.0, grads=grads)
    w = cnn.bf16_round(net.get_weights())
    flat = net.get_weights().astype(np.float64)
    sizes = [p.size for p in _params(w, dim)]
    # the biases are applied in FP32: exact in the reference
    p = _params(w, dim)
    for k in (1, 3, 5):
        at = sum(sizes[:k])
        p[k] = flat[at:at + sizes[k]].reshape(p[k].shape)
    z, (a0, z1, a1, z2, a2) = cnn.forward(np.moveaxis(x[..., :ci].astype(np.float64), -1, 1), p, bf16=True)
    rl, gz = cnn.bce_with_logits(z, y.reshape((tiles,) + (n,) * dim), 4.0)
    da2, dw3, db3 = cnn._conv_backward(a2, p[4], gz[:, None])
    da1, dw2, db2 = cnn._conv_backward(a1, p[2], da2 * (a2 > 0))
    _, dw1, db1 = cnn._conv_backward(a0, p[0], da1 * (a1 > 0))
    rg = [dw1, db1, dw2, db2, dw3, db3]
    assert loss.item() == pytest.approx(rl, rel=2e-2)
    got, at = grads.cpu().numpy().astype(np.float64), 0
    for r in rg:
        r = r.ravel()
        g = got[at:at + r.size]
        at += r.size
        assert np.linalg.norm(g - r) <= 2e-2 * np.linalg.norm(r), (at, np.linalg.norm(g - r) / np.linalg.norm(r))
    h.close()
