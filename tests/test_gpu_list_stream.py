"""The forward compositing's stream of depth ranks, at the sizes where it can
go wrong: full words (a row with every bit set, so that a word batch does not
fit the ring behind the batch in use), lists that end on, before and after a
batch of 64, and rows of several windows of 64 segments, most of them empty."""
import numpy as np
import pytest

from oracle import raster
from paper_2503_12886_amd import gbr, synth
from gpu_util import IMAGE_TOL, MASK_FRAC_MAX, compare_image, make_ctx, render

pytestmark = pytest.mark.gpu


def faint_pile(N, seed):
    """N splats that all cover a frame of one tile, none of them opaque: every
    bit of the tile's row is set and no pixel stops early."""
    rng = np.random.default_rng(seed)
    raw = np.zeros((N, 16), np.float32)
    raw[:, 0:2] = rng.normal(0.0, 1e-3, (N, 2))
    raw[:, 2] = rng.uniform(-0.05, 0.05, N)
    q = rng.normal(size=(N, 4))
    raw[:, 3:7] = q / np.linalg.norm(q, axis=1, keepdims=True)
    raw[:, 7:10] = rng.normal(-2.5, 0.1, (N, 3))
    raw[:, 10] = np.log(0.006 / 0.994) + rng.normal(0.0, 0.1, N)
    raw[:, 11:14] = rng.uniform(0.0, 1.0, (N, 3))
    return raw


@pytest.mark.parametrize("N", [1, 63, 64, 65, 256, 257, 900, 2100])
def test_full_rows(N):
    cam = synth.fixed_camera(16, 16, 18.75, 0.5, bg=(0.2, 0.3, 0.4))
    raw = faint_pile(N, N)
    ctx = make_ctx()
    imgs, _, _ = render(ctx, raw, [cam])
    ref, _, _, fl = raster.render(raw, cam)
    err, _ = compare_image(imgs[0], ref, fl, tag=f"full rows N={N}")
    assert err <= IMAGE_TOL
    last = int(gbr.gbr_inspect(ctx, "tile_last", 1)[0])
    part = gbr.gbr_inspect(ctx, "sorted_pass", N)
    full = gbr.gbr_inspect(ctx, "sorted", N)
    assert last > 0.9 * N and np.array_equal(part[:last], full[:last])
    ctx.close()


def test_sparse_rows_of_several_windows():
    """A row of 157 segments whose set bits sit in the first, a middle and the
    last of them: 80,000 splats in front of one tile's few."""
    N, cam = 80_000, synth.fixed_camera(48, 16, 18.75, 0.5)
    rng = np.random.default_rng(3)
    raw = faint_pile(N, 5)
    raw[:, 0] = -0.35 + rng.normal(0.0, 1e-3, N)         # over the first tile's left edge
    raw[:, 7:10] = -6.0
    raw[:, 2] = np.linspace(-0.05, 0.05, N)              # depth order = index order
    few = np.concatenate([np.arange(0, 40), np.arange(40_000, 40_030), np.arange(N - 70, N)])
    raw[few, 0] = 0.25
    raw[few, 7:10] = -4.0
    raw[few, 10] = -1.0
    ctx = make_ctx()
    imgs, _, _ = render(ctx, raw, [cam])
    ref, _, _, fl = raster.render(raw, cam)
    assert (fl != 0).mean() <= 2 * MASK_FRAC_MAX
    err, _ = compare_image(imgs[0], ref, fl, tag="sparse rows")
    assert err <= IMAGE_TOL
    ctx.close()
