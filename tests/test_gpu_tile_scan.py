"""The tile scan where it takes one block and one launch, and just past it:
tile counts on both sides of 4096, against the oracle's lists."""
import pytest

from oracle import raster
from paper_2503_12886_amd import gbr, synth
from gpu_util import make_ctx, render

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(16, 16), (1008, 1040), (1024, 1024), (272, 3856)])   # 1, 4095, 4096, 4097 tiles
def test_starts(w, h):
    cam = synth.fixed_camera(w, h, 1.17 * w, 0.5)
    raw = synth.make_scene(300, 0, seed=w)[0]
    ctx = make_ctx(max_pixels=1 << 21, max_entries=1 << 21)
    _, kept, images = render(ctx, raw, [cam])
    ranges, _, gauss, _ = raster.bin_and_sort([raster.project(raw, cam)], [cam], 16)
    n = ranges.shape[0]
    starts = gbr.gbr_inspect(ctx, "tile_start", n + 1)
    counts = ranges[:, 1] - ranges[:, 0]
    assert starts[0] == 0 and (starts[1:] - starts[:-1] == counts).all()
    assert (gbr.gbr_inspect(ctx, "sorted", int(starts[-1])) == gauss).all()
    del kept, images
    ctx.close()
