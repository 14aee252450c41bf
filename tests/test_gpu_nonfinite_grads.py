"""An image gradient that is not finite at one pixel (or overflows against a
colour): a Gaussian that the pixel did not take keeps its position, rotation,
scale and opacity gradients, bit for bit those with a zero there; those that
it took lose theirs."""
import numpy as np
import pytest

from oracle import raster
from paper_2503_12886_amd import gbr, synth
from gpu_util import dev, host, make_ctx, render

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("value", [np.nan, np.inf, 3e38])
def test_one_pixel(tile, value):
    import torch
    N, cam = 60, synth.fixed_camera(40, 24, 40.0, 0.5, bg=(0.2, 0.3, 0.4))
    rng = np.random.default_rng(3)
    raw = np.zeros((N, 16), np.float32)
    raw[:, 0] = rng.uniform(-0.2, 0.2, N)
    raw[:, 1] = rng.uniform(-0.12, 0.12, N)
    raw[:, 2] = rng.uniform(-0.05, 0.05, N)
    raw[:, 3:7] = rng.normal(size=(N, 4))
    raw[:, 7:10] = rng.uniform(-4.5, -3.5, (N, 3))
    raw[:, 10] = rng.uniform(-2.0, 1.0, N)
    raw[:, 11:14] = rng.uniform(2.0, 3.0, (N, 3))          # (3e38 of them is infinite)
    _, _, nc, fl = raster.render(raw, cam)
    lists, _ = raster.contributors(raw, cam)
    ok = np.argwhere((fl == 0) & (nc >= 3))
    y, x = ok[len(ok) // 2]
    takes = np.zeros(N, bool)
    takes[lists[y, x, :nc[y, x]]] = True
    ctx = make_ctx(tile=tile)
    _, blended, images = render(ctx, raw, [cam])           # (the pass reads the blended Gaussians again)
    dimg = rng.normal(size=(3, cam.height, cam.width)).astype(np.float32)
    draws = []
    for v in (0.0, value):
        dimg[:, y, x] = v
        draw = torch.zeros(N * 16, device="cuda")
        gbr.gbr_render_backward(ctx, dev(dimg.ravel()), draw)
        draws.append(host(draw).reshape(N, 16)[:, :11])
    assert np.isfinite(draws[0]).all() and 3 <= takes.sum() < N // 2
    assert np.array_equal(draws[0][~takes], draws[1][~takes])
    assert not np.isfinite(draws[1][takes]).all()
    ctx.close()
