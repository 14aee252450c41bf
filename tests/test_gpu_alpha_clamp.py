"""The clamp of alpha at 0.99 is exact: behind black splats that are opaque
over the whole frame a white background shows through by the float32 products
of 1 - 0.99, bit for bit, whatever the splat's own opacity above it."""
import numpy as np
import pytest

from paper_2503_12886_amd import synth
from gpu_util import make_ctx, render

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("logit", [5.0, 8.0, 30.0])     # opacity 0.9933, 0.99966, 1
def test_clamp(tile, logit):
    cam = synth.fixed_camera(24, 20, 18.75, 0.5, bg=(1.0, 1.0, 1.0))
    ctx = make_ctx(tile=tile)
    t = np.float32(1.0)
    a = np.float32(0.99)
    for n in (1, 2):                                    # a third would stop the pixel
        raw = np.zeros((n, 16), np.float32)
        raw[:, 3] = 1.0                                 # a power of -4e-4 at the corner
        raw[:, 7:10] = 3.0
        raw[:, 2] = np.linspace(0.0, 0.01, n)
        raw[:, 10] = logit
        t = np.float32(np.float64(t) * (1.0 - np.float64(a)))   # one rounding, as fma(-a, t, t)
        imgs, _, _ = render(ctx, raw, [cam])
        if n == 2 and t < 1e-4:                         # 1e-4 less a rounding: the second stops the pixel
            t = np.float32(np.float64(1.0) - np.float64(a))
        assert (imgs[0] == t).all(), (n, imgs[0].min(), imgs[0].max(), t)
    ctx.close()
