"""A batch's frame table passed as kernel arguments (up to 16 frames) and
uploaded (17): every frame's image is the bits of the frame rendered alone,
with the batches in turn on one context."""
import numpy as np
import pytest

from paper_2503_12886_amd import synth
from gpu_util import make_ctx, render

pytestmark = pytest.mark.gpu


def test_frames():
    cams = synth.make_cameras(17, resolutions=[(48, 32), (33, 50), (16, 16)], yaw_deg=30.0, dist=(0.4, 0.7))
    raws = [synth.make_scene(40 + 3 * b, 0, seed=b)[0] for b in range(17)]
    ctx = make_ctx(max_frames=17, max_pixels=1 << 16, max_entries=1 << 18)
    alone = [render(ctx, raws[b], [cams[b]])[0][0] for b in range(17)]
    for B in (16, 17, 2, 17, 16):
        offsets = np.concatenate([[0], np.cumsum([r.shape[0] for r in raws[:B]])]).tolist()
        imgs, _, _ = render(ctx, np.concatenate(raws[:B]), cams[:B], offsets)
        for b in range(B):
            assert (imgs[b] == alone[b]).all(), (B, b)
    ctx.close()
