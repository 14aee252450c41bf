"""The two forms of the splats' gradient sums: a batch of 500000 splats or more
takes the two-launch form, its frames one by one the one-launch form, which the
other tests hold against the oracle.  Both add a splat's partials in the same
order and chain them in float64, so a row differs by a float32 rounding at
most: 2^-23 of its value, with a floor of 1e-9 of the frame's largest (float64
roundings under cancellation)."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr, synth
from gpu_util import dev, host, make_ctx, render
from test_gpu_list_stream import faint_pile

pytestmark = pytest.mark.gpu


def backward(ctx, raw, cams, offsets, dimg, total):
    import torch
    _, kept, images = render(ctx, raw, cams, offsets)     # (the pass reads the blended Gaussians again)
    draw = torch.full((total * 16,), float("nan"), device="cuda")
    gbr.gbr_render_backward(ctx, dev(dimg), draw)
    out = host(draw).reshape(total, 16)
    del kept, images
    return out


# the crowd's size puts the batch just below, on and above the line
@pytest.mark.parametrize("tile", [8, 32])
@pytest.mark.parametrize("total", [499999, 500000, 500257])
def test_forms(total, tile):
    # frames of 64 and fewer splats, around a workgroup's 256, a pile whose
    # waves hold a few thousand flagged entries each, and a crowd
    sizes = [1, 63, 65, 255, 256, 257, 300, 130]
    sizes.append(total - sum(sizes))
    cams = [synth.fixed_camera(64, 64, 75.0, 0.5, bg=(0.2, 0.3, 0.4)) for _ in sizes]
    raws = [synth.make_scene(n, 0, seed=n)[0] for n in sizes]
    raws[6] = faint_pile(300, 5)                     # in all 64 or 4 tiles, no pixel stops
    raws[6][:, 7:11] += 1.0
    raws[7] = faint_pile(130, 6)
    raws[7][:, 2] += np.where(np.arange(130) % 3 == 0, -1.0, 0.0).astype(np.float32)   # a third behind the camera
    offsets = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    rng = np.random.default_rng(total)
    dimgs = [rng.normal(size=3 * 64 * 64).astype(np.float32) for _ in sizes]
    ctx = make_ctx(tile=tile, max_pixels=1 << 16, max_entries=1 << 22)
    for again in range(2):                           # the flags were left cleared
        got = backward(ctx, np.concatenate(raws), cams, offsets, np.concatenate(dimgs), total)
        for b, n in enumerate(sizes):
            ref = backward(ctx, raws[b], cams[b:b + 1], [0, n], dimgs[b], n)
            mine = got[offsets[b]:offsets[b + 1]]
            assert np.isfinite(mine).all()
            bound = 2.0 ** -23 * np.abs(ref) + 1e-9 * np.abs(ref).max()
            assert (np.abs(mine - ref) <= bound).all(), (b, n, np.abs(mine - ref).max(), np.abs(ref).max())
    assert np.abs(got[offsets[6]:offsets[7], 10]).min() > 0   # every splat of the pile has a gradient
    ctx.close()
