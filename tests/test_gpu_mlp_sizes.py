"""The weights MLP's two forms (all weights held in registers up to 64 inputs
and 256 hidden units, layer by layer beyond) at the edges of both and of the
units a wave forms together, against a float64 evaluation.  A unit's sum of n
products, in any order, is within (n + 2) u of its terms' magnitudes (Higham,
section 3.1), and a layer's input errors reach the next through its weights'
magnitudes; the bound below carries both through the three layers."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr, synth
from gpu_util import U32, dev, host, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,hidden,K,B", [(1, 1, 1, 1), (56, 256, 20, 16), (63, 255, 3, 2), (64, 256, 64, 3),
                                             (65, 256, 20, 2), (64, 257, 17, 2), (300, 513, 33, 3), (1024, 1024, 64, 1),
                                             (7, 16, 4, 5), (64, 15, 5, 4)])
def test_forward(d_in, hidden, K, B):
    import torch
    p = synth.make_mlp(K=K, seed=d_in + K, d_in=d_in, hidden=hidden)
    theta = np.random.default_rng(B).normal(size=(B, d_in)).astype(np.float32)
    flat = np.concatenate([p[n].ravel() for n in ("W1", "b1", "W2", "b2", "W3", "b3")]).astype(np.float32)
    ctx = make_ctx()
    psi = torch.full((B, K), float("nan"), device="cuda")
    gbr.gbr_mlp_forward(ctx, dev(flat), dev(theta), d_in, hidden, K, psi)
    x, err = theta.astype(np.float64), np.zeros((B, d_in))
    for i in (1, 2, 3):
        W, b = p[f"W{i}"].astype(np.float64), p[f"b{i}"].astype(np.float64)
        n = x.shape[1] + 2
        err = err @ np.abs(W).T + n * U32 / (1 - n * U32) * ((np.abs(x) + err) @ np.abs(W).T + np.abs(b))
        x = x @ W.T + b
        if i < 3:
            x = np.maximum(x, 0.0)
    assert np.all(np.abs(host(psi) - x) <= err)
    ctx.close()
