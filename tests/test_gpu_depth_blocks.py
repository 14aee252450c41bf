"""The depth order over the bucket passes' blocks of 8192 splats: frames of one
to three blocks, ends on and beside a block's, in one batch with frames that
use fewer blocks and other bucket counts; depths spread evenly, all in a few
buckets, and some behind the camera."""
import numpy as np
import pytest

from oracle import raster
from paper_2503_12886_amd import gbr, synth
from gpu_util import make_ctx, render
from test_gpu_list_stream import faint_pile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [8191, 40], [8192], [3, 8193, 700], [16385, 1, 8192, 20000, 511, 513],
                                   [8193] * 8, [600] * 14, [100] * 15 + [99]])    # (frames on XCDs of their own)
@pytest.mark.parametrize("spread", ["even", "clustered"])
def test_order(sizes, spread):
    rng = np.random.default_rng(sum(sizes))
    raws = []
    for n in sizes:
        raw = faint_pile(n, n)
        z = rng.permutation(n) * 1e-5                       # steps of more than a float32 at these depths
        if spread == "clustered":
            z = np.where(rng.uniform(size=n) < 0.9, 1e-6 * rng.permutation(n), z + 0.1)
        raw[:, 2] = z
        raw[::7, 2] -= 2.0 if n > 1 else 0.0                # behind the camera
        raws.append(raw)
    cams = [synth.fixed_camera(16, 16, 18.75, 0.5) for _ in sizes]
    # the oracle's lists (one tile a frame)
    ranges, frame, gauss, _ = raster.bin_and_sort([raster.project(r, c) for r, c in zip(raws, cams)], cams, 16)
    base = np.concatenate([[0], np.cumsum(sizes)])
    ctx = make_ctx(max_pixels=1 << 14, max_entries=1 << 18)
    _, kept, images = render(ctx, np.concatenate(raws), cams, base.tolist())
    starts = gbr.gbr_inspect(ctx, "tile_start", len(sizes) + 1).astype(np.int64)
    got = gbr.gbr_inspect(ctx, "sorted", int(starts[-1]))
    assert (starts[:-1] == ranges[:, 0]).all() and starts[-1] == ranges[-1, 1]
    assert (got == base[frame] + gauss).all()
    del kept, images
    ctx.close()
