"""The contraction for the weights around the sizes where a wave takes several spans
(1024 workgroups of 64 Gaussians, half as many again for at most 16 frames and
32 slices), against float64 within the summation bound of its order."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr
from gpu_util import check_sum_bound, dev, host, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,K", [(3, 5), (16, 32), (17, 5), (3, 33)])
@pytest.mark.parametrize("blocks", [1024, 1025, 1536, 1537])
def test_line(B, K, blocks):
    import torch
    N = 64 * blocks - 7
    rng = np.random.default_rng(B + K + blocks)
    bases = rng.normal(size=(K + 1, N, 16)).astype(np.float32)
    draw = rng.normal(size=(B, N, 16)).astype(np.float32)
    draw[..., 14:] = 0.0
    ctx = make_ctx(max_splats=N * B)
    dw = torch.zeros(B, K, device="cuda")
    gbr.gbr_blend_backward(ctx, dev(draw), dev(bases), dev(np.zeros((B, K), np.float32)), None, dw)
    d, s = draw[..., :14].reshape(B, -1).astype(np.float64), bases[1:, :, :14].reshape(K, -1).astype(np.float64)
    # a product, at most 255 additions in a span, the wave's spans, 4 waves, the
    # partials' 16-tree, their passes and the 64-tree
    spans = -(-N * 16 // 256)
    depth = 1 + 255 + -(-spans // 4096) + 3 + 4 + 2 + 6
    check_sum_bound(host(dw), d @ s.T, np.abs(d) @ np.abs(s).T, depth, N * 14, f"dweights B={B} K={K} blocks={blocks}")
    ctx.close()
