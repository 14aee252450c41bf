"""The gradient written over the Gaussians that were rendered, below and past the
size that takes two launches, against one written elsewhere: the same sums
in the same order chained in float64, so a float32 rounding apart (2^-23 of a
value, with a floor of 1e-9 of the frame's largest)."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr, synth
from gpu_util import dev, host, make_ctx, render

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1000, 300), (499_000, 257, 743), (3000, 500_100)])
def test_in_place(sizes):
    import torch
    total = sum(sizes)
    cams = [synth.fixed_camera(64, 64, 75.0, 0.5) for _ in sizes]
    raw = np.concatenate([synth.make_scene(n, 0, seed=n)[0] for n in sizes])
    offsets = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    dimg = dev(np.random.default_rng(total).normal(size=3 * 64 * 64 * len(sizes)).astype(np.float32))
    ctx = make_ctx(max_pixels=1 << 16, max_entries=1 << 22)
    _, rendered, images = render(ctx, raw, cams, offsets)
    draw = torch.full_like(rendered, float("nan"))
    gbr.gbr_render_backward(ctx, dimg, draw)
    gbr.gbr_render_backward(ctx, dimg, rendered)
    a, b = host(draw).reshape(total, 16), host(rendered).reshape(total, 16)
    for i in range(len(sizes)):
        x, y = a[offsets[i]:offsets[i + 1]], b[offsets[i]:offsets[i + 1]]
        assert np.abs(x).max() > 0
        assert (np.abs(x - y) <= 2.0 ** -23 * np.abs(x) + 1e-9 * np.abs(x).max()).all()
    ctx.close()
