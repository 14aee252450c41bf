"""The backward compositing's groups: a quadrant that takes 1 to a few more
than 8 entries of a batch (short groups), lists that end on, before and after
a batch of 64, at the tiles that take the sums 8 entries at a time and at the
one that does not, frames that leave part of their last tiles empty."""
import numpy as np
import pytest

from oracle import raster
from paper_2503_12886_amd import gbr, synth
from gpu_util import dev, grad_check, host, make_ctx, render, zero_flagged
from test_gpu_list_stream import faint_pile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("N", [1, 2, 7, 8, 9, 63, 64, 65, 130])
def test_groups(tile, N):
    import torch
    cam = synth.fixed_camera(21, 13, 18.75, 0.5, bg=(0.2, 0.3, 0.4))
    raw = faint_pile(N, N + tile)
    raw[:, 10] += 3.0                               # opacities around 0.1
    raw[::3, 0:2] += 0.12                           # some over one quadrant only
    raw[::3, 7:10] -= 1.0
    ctx = make_ctx(tile=tile)
    imgs, blended, images = render(ctx, raw, [cam])   # (the pass reads the blended Gaussians again)
    _, _, nc, fl = raster.render(raw, cam)
    dimg = np.random.default_rng(N).normal(size=(3, cam.height, cam.width)).astype(np.float32)
    dimg = zero_flagged([dimg], [fl])[0]
    draw = torch.zeros(N * 16, device="cuda")
    gbr.gbr_render_backward(ctx, dev(dimg.ravel()), draw)
    got = host(draw).reshape(N, 16)
    ref, _ = raster.render_grad(raw, cam, dimg)
    mag = raster.adjoint_magnitude(raw, cam, dimg)
    rel, worst = grad_check(got[:, :14], ref[:, :14], tag=f"groups N={N} tile={tile}", mag=mag[:, :14], n_max=nc.max())
    assert rel <= 1e-3 and worst <= 1.0, (rel, worst)
    ctx.close()
