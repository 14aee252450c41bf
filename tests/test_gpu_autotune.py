"""The autotuner times what differs: at tiles of 8 and 16 pixels, where the chunk
makes no difference, one time stands for the three chunks, and the pick's
chunk there is always the first."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr, synth
from gpu_util import dev, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [40, 136])
def test_times(size):
    import torch
    N, cam = 3000, synth.fixed_camera(size, size, 1.2 * size, 0.5)
    raw = dev(synth.make_scene(N, 0, seed=1)[0])
    ctx = make_ctx(tile=8, chunk=256)
    images = torch.zeros(3 * size * size, device="cuda")
    dimages, draw = torch.ones_like(images), torch.zeros(N * 16, device="cuda")
    tile, chunk, times = gbr.gbr_autotune(ctx, raw, [0, N], [cam], images, dimages, draw)
    assert all(t > 0 for t in times)
    assert times[0] == times[1] == times[2] and times[3] == times[4] == times[5]
    assert (tile, chunk) == [(t, c) for t in (8, 16, 32) for c in (64, 128, 256)][int(np.argmin(np.float32(times)))]
    assert chunk == 64 or tile == 32
    ctx.close()
